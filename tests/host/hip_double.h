// A HIP runtime for host tests of the library's runtime code (contexts, streams,
// the block cache): the test program defines the runtime's entry points itself,
// and the dynamic linker binds the library's calls to the program's symbols, so
// libigafd.so runs as it is built without a GPU.  Device memory is reserved
// address space (only touched where something small is copied or cleared),
// kernels are not run, and what the library asks of the runtime is recorded.
#pragma once

#include <hip/hip_runtime_api.h>
#include <sys/mman.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace hip_double {

struct Alloc {
  size_t bytes;
  int device;
};
struct Sync {
  int device;          // device current at the call
  hipStream_t stream;  // the stream waited for; kWhole: the whole device
};
struct Attr {
  const void* fn;
  int value;
};
inline const hipStream_t kWhole = (hipStream_t)-1;

inline std::recursive_mutex mu;
inline thread_local int inside = 0;    // this thread is in the runtime: its allocations are not the library's
struct Locked {
  Locked() {
    mu.lock();
    inside += 1;
  }
  ~Locked() {
    inside -= 1;
    mu.unlock();
  }
};
inline std::map<void*, Alloc> live;    // device allocations
inline size_t used[2] = {0, 0};        // their bytes per device
inline size_t capacity = (size_t)288 << 30;
inline long long large_mallocs = 0, frees = 0;  // of 1 MiB and more; all
inline std::vector<Sync> syncs;
inline std::vector<Attr> attrs;        // hipFuncSetAttribute, dynamic LDS
inline int cus = 256;
inline long long device_allocs = 0, fail_alloc = -1;  // with fail_alloc >= 0, that one and the next fail
inline bool over_limit = false;        // a launch asked for more dynamic LDS than its function's limit
inline hipStream_t dead = nullptr;     // a stream that was destroyed: waiting for it fails
inline bool device_lost = false;       // waiting for the device fails too
inline thread_local int device = 0;
inline thread_local hipError_t last = hipSuccess;

inline hipError_t done(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
constexpr size_t kTouch = 1 << 16;     // larger ranges are not copied or cleared

inline size_t room_from(const void* p) {  // bytes from p to the end of its allocation (0: not device memory)
  auto it = live.upper_bound(const_cast<void*>(p));
  if (it == live.begin()) return 0;
  --it;
  const char* b = (const char*)it->first;
  return (const char*)p < b + it->second.bytes ? (size_t)(b + it->second.bytes - (const char*)p) : 0;
}

// live device bytes of a device
inline size_t bytes_on(int d) {
  Locked lock;
  return used[d];
}
inline void forget() {
  Locked lock;
  syncs.clear();
  attrs.clear();
  large_mallocs = frees = 0;
}

}  // namespace hip_double

extern "C" {

using namespace hip_double;

hipError_t hipGetDevice(int* d) {
  *d = device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  if (d < 0 || d > 1) return done(hipErrorInvalidDevice);
  device = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? cus : 160 * 1024;  // the others asked for are LDS sizes
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}

hipError_t hipMalloc(void** p, size_t bytes) {
  Locked lock;
  *p = nullptr;
  const long long k = device_allocs++;
  if (fail_alloc >= 0 && (k == fail_alloc || k == fail_alloc + 1)) return done(hipErrorOutOfMemory);
  if (used[device] + bytes > capacity) return done(hipErrorOutOfMemory);
  void* m = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (m == MAP_FAILED) return done(hipErrorOutOfMemory);
  live[m] = Alloc{bytes, device};
  used[device] += bytes;
  large_mallocs += bytes >= (1 << 20);
  *p = m;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  Locked lock;
  if (!p) return hipSuccess;
  const auto it = live.find(p);
  if (it == live.end()) return done(hipErrorInvalidValue);
  munmap(p, it->second.bytes);
  used[it->second.device] -= it->second.bytes;
  live.erase(it);
  frees += 1;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int) {
  *p = std::calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  std::free(p);
  return hipSuccess;
}

// ranges outside the allocation they start in are reported as errors
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  Locked lock;
  for (const void* p : {(const void*)d, s}) {
    const size_t room = room_from(p);
    if (room && n > room) return done(hipErrorInvalidValue);
  }
  if (n <= kTouch) std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  return hipMemcpy(d, s, n, k);
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  Locked lock;
  if (n > room_from(d)) return done(hipErrorInvalidValue);
  if (n <= kTouch) std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemset2DAsync(void* d, size_t pitch, int, size_t w, size_t h, hipStream_t) {
  Locked lock;
  if (h > 0 && (h - 1) * pitch + w > room_from(d)) return done(hipErrorInvalidValue);
  return hipSuccess;
}

hipError_t hipStreamSynchronize(hipStream_t s) {
  Locked lock;
  if (dead && s == dead) return done(hipErrorContextIsDestroyed);
  syncs.push_back(Sync{device, s});
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
  Locked lock;
  if (device_lost) return done(hipErrorLaunchFailure);
  syncs.push_back(Sync{device, kWhole});
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int) {
  *s = (hipStream_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::free(s);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = (hipEvent_t)std::malloc(1);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* fn, hipFuncAttribute a, int v) {
  Locked lock;
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) attrs.push_back(Attr{fn, v});
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void**, size_t lds, hipStream_t) {
  Locked lock;
  size_t limit = 64 * 1024;
  for (const Attr& a : attrs)
    if (a.fn == fn) limit = (size_t)a.value;
  if (lds > limit) over_limit = true;
  return hipSuccess;
}

}  // extern "C"
