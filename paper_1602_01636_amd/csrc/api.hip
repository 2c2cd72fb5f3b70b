// C ABI: setup, sizes, load vector, A product, preconditioner apply, PCG solve.
//
// The conjugate gradient method with the SPD preconditioner P (paper Sec. 3)
// runs as a stream of device kernels whose scalars (rho, p^T A p, alpha,
// beta, ||r||^2) live in device memory.  Every kernel of an iteration checks a
// device stop flag first, so the host enqueues several iterations ahead and
// reads the state back only every `check_every` iterations; iterations
// enqueued past convergence are no-ops.  Reductions are per-block partial sums
// finished by one block in a fixed order, so results are bitwise reproducible.
//
// Stopping rule (the paper states none): x0 = 0 unless given, stop when
// ||r_k||_2 <= rtol ||b||_2 on the recursive residual; then the true residual
// b - A x is evaluated in FP64 and the iteration restarts from it if it does
// not meet the tolerance.  flexible = 1 uses the Polak-Ribiere beta
// (r_{k+1}, z_{k+1} - z_k) / (r_k, z_k) for inexact (FP32/BF16) applies.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <unordered_map>

#include "internal.h"
#include "reduce.h"

namespace igafd {

namespace {
thread_local std::string g_err;
}

void set_error(const std::string& msg) { g_err = msg; }

namespace {
// the body of a call that allocates host memory: none leaves the C interface as an exception
template <class F>
igafd_status guarded(const F& body) {
  try {
    return body();
  } catch (const std::exception&) {
    try {
      set_error("out of host memory");
    } catch (const std::exception&) {
    }
    return IGAFD_ERR_ALLOC;
  }
}
}  // namespace

// Device blocks of 1 MiB or more, kept for the next context when one is
// released.  Returning gigabytes to the driver and taking them again costs a
// clear of that memory at about 33 GB/s once a process has cycled through its
// cleared reserve (about 140 GB): 130 ms for the 4.3 GB band of a 112^3, p = 4
// problem whose setup takes 20.  Bounds: kCacheBytes per device; a block is
// reused for requests of at least 4/5 of its size, and given back to the
// driver when kCacheAge later requests found no use for it, when the bound is
// exceeded (oldest first), when an allocation of this library fails, or by
// igafd_release_cached (a process that makes no further request keeps its
// blocks until it calls that).  Callers release a block only after the work
// that used it has finished.
namespace {
constexpr size_t kCacheMin = 1u << 20, kCacheBytes = (size_t)8 << 30;
constexpr long long kCacheAge = 64;
struct Block {
  void* p;
  size_t bytes;
  int device;
  long long stamp;
};
// (never destroyed: contexts may outlive the library's static objects)
std::mutex& g_block_mutex = *new std::mutex;
std::vector<Block>& g_cached = *new std::vector<Block>;                              // oldest first
std::unordered_map<void*, Block>& g_blocks = *new std::unordered_map<void*, Block>;  // in use
long long g_block_clock = 0;

bool record_block(const Block& b) {  // under the mutex
  try {
    g_blocks[b.p] = b;
  } catch (const std::bad_alloc&) {
    return false;
  }
  return true;
}

void trim_blocks(int device, size_t keep, long long oldest) {  // under the mutex
  size_t held = 0;
  for (const Block& b : g_cached) held += b.device == device ? b.bytes : 0;
  for (size_t k = 0; k < g_cached.size();) {
    const Block b = g_cached[k];
    if ((b.device == device && held > keep) || b.stamp < oldest) {
      (void)hipFree(b.p);
      if (b.device == device) held -= b.bytes;
      g_cached.erase(g_cached.begin() + (long)k);
    } else {
      ++k;
    }
  }
}
}  // namespace

// the cached blocks of the current device go back to the driver
static void drop_blocks() {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return;
  std::lock_guard<std::mutex> lock(g_block_mutex);
  trim_blocks(device, 0, g_block_clock - kCacheAge);
}

hipError_t device_malloc(void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    drop_blocks();
    e = hipMalloc(p, bytes);
  }
  return e;
}

igafd_status block_alloc(void** p, size_t bytes) {
  *p = nullptr;
  int device = 0;
  IGAFD_HIP_CHECK(hipGetDevice(&device));
  if (bytes >= kCacheMin) {
    std::lock_guard<std::mutex> lock(g_block_mutex);
    g_block_clock += 1;
    size_t best = g_cached.size();
    for (size_t k = 0; k < g_cached.size(); ++k) {
      const Block& b = g_cached[k];
      if (b.device == device && b.bytes >= bytes && b.bytes - bytes <= bytes / 4 &&
          (best == g_cached.size() || b.bytes < g_cached[best].bytes))
        best = k;
    }
    if (best < g_cached.size() && record_block(g_cached[best])) {
      *p = g_cached[best].p;
      g_cached.erase(g_cached.begin() + (long)best);
    }
    trim_blocks(device, kCacheBytes, g_block_clock - kCacheAge);
    if (*p) return IGAFD_OK;
  }
  const hipError_t e = device_malloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
    set_error(std::string("device allocation of ") + std::to_string(bytes) + " bytes: " + hipGetErrorString(e));
    return IGAFD_ERR_HIP;
  }
  if (bytes >= kCacheMin) {
    std::lock_guard<std::mutex> lock(g_block_mutex);
    (void)record_block(Block{*p, bytes, device, 0});  // one without a record is not kept later
  }
  return IGAFD_OK;
}

// Waits for a stream of a device, which need not be the current one (the null
// stream is each device's own).  A stream that its owner has destroyed leaves
// only the device to wait for.
bool wait_stream(hipStream_t stream, int device) {
  int current = device;
  (void)hipGetDevice(&current);
  if (current != device && hipSetDevice(device) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  hipError_t e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    e = hipDeviceSynchronize();
    (void)hipGetLastError();  // the failed wait is no later call's error
  }
  if (current != device) (void)hipSetDevice(current);
  return e == hipSuccess;
}

void block_free(void* p, bool idle) {
  if (!p) return;
  {
    std::lock_guard<std::mutex> lock(g_block_mutex);
    const auto it = g_blocks.find(p);
    if (it != g_blocks.end()) {
      Block b = it->second;
      g_blocks.erase(it);
      if (!idle) {
        (void)hipFree(p);
        return;
      }
      b.stamp = g_block_clock;
      try {
        g_cached.push_back(b);
      } catch (const std::bad_alloc&) {
        (void)hipFree(p);
        return;
      }
      trim_blocks(b.device, kCacheBytes, g_block_clock - kCacheAge);
      return;
    }
  }
  (void)hipFree(p);
}

// Block partials every reduction of a context may write (per sum): the
// vector kernels' grid, every FD path and tile count, and at least 1025 (the
// spectral bounds' blocks plus their result).
int partial_capacity(const igafd_ctx* c) {
  const int vb = (int)((c->N + kBlock - 1) / kBlock);
  return std::max(std::max(vb, 1025), fd_dot_blocks_max(c));
}

namespace {

enum { RED_BB_RR = 0, RED_PQ = 1, RED_RR = 2, RED_RZ = 3, RED_RHO0 = 4, RED_TRUE = 5 };
constexpr int kHistDefault = 2001;  // history entries allocated with the workspace

// r = b - y (y = A x0, or r = b when y is null); x = 0 unless keep_x.
// Partials: (b, b) and (r, r).
__global__ __launch_bounds__(kBlock) void k_init(const double* __restrict__ b, const double* __restrict__ y,
                                                 double* __restrict__ r, double* __restrict__ x, int keep_x,
                                                 long long N, double* __restrict__ partial) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  double bb = 0.0, rr = 0.0;
  if (i < N) {
    const double bi = b[i];
    const double ri = y ? bi - y[i] : bi;
    r[i] = ri;
    if (!keep_x) x[i] = 0.0;
    bb = bi * bi;
    rr = ri * ri;
  }
  block_sum2(bb, rr);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = bb;
    partial[gridDim.x + blockIdx.x] = rr;
  }
}

// Grouped start of batched solves: r = b, x = 0, partials (b, b), (r, r);
// and r = b - q with the partials (r, r) of the true residual.
struct InitJob {
  const double* b;
  const double* q;  // null: r = b, x = 0 (start); else r = b - q (true residual)
  double* r;
  double* x;
  long long N;
  double* partial;
  int gx;
};

__global__ __launch_bounds__(kBlock) void k_init_g(const InitJob* __restrict__ jobs, const int* __restrict__ start,
                                                   int njobs) {
  const int j = group_job(start, njobs, (int)blockIdx.x);
  const InitJob& t = jobs[j];
  const int bx = (int)blockIdx.x - start[j];
  const long long i = (long long)bx * kBlock + threadIdx.x;
  double bb = 0.0, rr = 0.0;
  if (i < t.N) {
    const double bi = t.b[i];
    const double ri = t.q ? bi - t.q[i] : bi;
    t.r[i] = ri;
    if (!t.q) t.x[i] = 0.0;
    bb = bi * bi;
    rr = ri * ri;
  }
  if (t.q) {
    const double s = block_sum(rr);
    if (threadIdx.x == 0) t.partial[bx] = s;
  } else {
    block_sum2(bb, rr);
    if (threadIdx.x == 0) {
      t.partial[bx] = bb;
      t.partial[t.gx + bx] = rr;
    }
  }
}

// dst = src over N values per job (into the zero-halo buffers)
struct CopyJob {
  const double* src;
  double* dst;
  long long N;
};

__global__ __launch_bounds__(kBlock) void k_copy_g(const CopyJob* __restrict__ jobs, const int* __restrict__ start,
                                                   int njobs) {
  const int j = group_job(start, njobs, (int)blockIdx.x);
  const CopyJob& t = jobs[j];
  const long long i = (long long)((int)blockIdx.x - start[j]) * kBlock + threadIdx.x;
  if (i < t.N) t.dst[i] = t.src[i];
}

// One block: sum partial[0..count) (and partial[count..2 count) when two
// sums are pending) in a fixed order, then the scalar step of CG.
constexpr int kReduceBlock = 1024;  // one wide block: a few independent loads per thread

__device__ __forceinline__ void reduce_body(const double* __restrict__ partial, int count, int two, int which,
                                            SolverState* __restrict__ s, double* __restrict__ hist) {
  if (which != RED_BB_RR && which != RED_RHO0 && which != RED_TRUE && s->flag != FLAG_RUNNING) return;
  double a = 0.0, b = 0.0;
#pragma unroll 4
  for (int k = threadIdx.x; k < count; k += kReduceBlock) {
    a += partial[k];
    if (two) b += partial[count + k];
  }
  block_sum2<kReduceBlock>(a, b);
  if (threadIdx.x != 0) return;
  switch (which) {
    case RED_BB_RR:  // a = (b,b), b = (r,r)
      s->bb = a;
      s->tol2 = s->tol2 * a;  // tol2 holds rtol^2 on entry
      s->rr = b;
      s->iters = 0;
      s->flag = (b <= s->tol2) ? FLAG_CONVERGED : FLAG_RUNNING;
      if (hist && s->hist_cap > 0) hist[0] = a > 0.0 ? sqrt(b / a) : 0.0;
      break;
    case RED_RHO0:
      s->rho = a;
      break;
    case RED_PQ: {
      s->pq = a;
      if (!(a > 0.0) || !isfinite(a) || !isfinite(s->rho)) {
        s->flag = FLAG_BREAKDOWN;
      } else {
        s->alpha = s->rho / a;
        s->iters += 1;
      }
      break;
    }
    case RED_RR:  // a = (r,r), b = (r, z_old) for the flexible form
      s->rr = a;
      s->rzold = b;
      // restarts and the plain-P fallback run past maxit: write only what the
      // caller's maxit+1 entries hold
      if (hist && s->iters < s->hist_cap) hist[s->iters] = s->bb > 0.0 ? sqrt(a / s->bb) : 0.0;
      if (a <= s->tol2)
        s->flag = FLAG_CONVERGED;
      else if (!isfinite(a))
        s->flag = FLAG_BREAKDOWN;
      else if (s->iters >= s->maxit)
        s->flag = FLAG_MAXIT;
      break;
    case RED_RZ: {
      s->rz = a;
      s->beta = s->flexible ? (a - s->rzold) / s->rho : a / s->rho;
      s->rho = a;
      break;
    }
    case RED_TRUE:
      s->rrtrue = a;
      break;
  }
}

__global__ __launch_bounds__(kReduceBlock) void k_reduce(const double* __restrict__ partial, int count, int two,
                                                         int which, SolverState* __restrict__ s,
                                                         double* __restrict__ hist) {
  reduce_body(partial, count, two, which, s, hist);
}

// Grouped forms of the CG kernels (batched solves): one launch runs the step
// for several problems; job j owns blocks [start[j], start[j+1]) (one block
// per job for the reductions).
struct ReduceJob {
  const double* partial;
  int count, two;
  SolverState* s;
};

__global__ __launch_bounds__(kReduceBlock) void k_reduce_g(const ReduceJob* __restrict__ jobs, int which) {
  const ReduceJob& t = jobs[blockIdx.x];
  reduce_body(t.partial, t.count, t.two, which, t.s, nullptr);
}

// x += alpha p; r -= alpha q; partials (r, r) and (r, z_old).
__device__ __forceinline__ void update_xr_body(double* __restrict__ x, double* __restrict__ r,
                                               const double* __restrict__ p, const double* __restrict__ q,
                                               const double* __restrict__ zold, const SolverState* __restrict__ s,
                                               long long N, double* __restrict__ partial, int bx, int gx) {
  const double alpha = s->alpha;
  const long long i = (long long)bx * kBlock + threadIdx.x;
  double rr = 0.0, rz = 0.0;
  if (i < N) {
    x[i] = fma(alpha, p[i], x[i]);
    const double ri = fma(-alpha, q[i], r[i]);
    r[i] = ri;
    rr = ri * ri;
    if (zold) rz = ri * zold[i];
  }
  block_sum2(rr, rz);
  if (threadIdx.x == 0) {
    partial[bx] = rr;
    partial[gx + bx] = rz;
  }
}

__global__ __launch_bounds__(kBlock) void k_update_xr(double* __restrict__ x, double* __restrict__ r,
                                                      const double* __restrict__ p, const double* __restrict__ q,
                                                      const double* __restrict__ zold, const SolverState* __restrict__ s,
                                                      long long N, double* __restrict__ partial) {
  if (s->flag != FLAG_RUNNING) return;
  update_xr_body(x, r, p, q, zold, s, N, partial, (int)blockIdx.x, (int)gridDim.x);
}

struct UpdateXrJob {
  double* x;
  double* r;
  const double* p;
  const double* q;
  const double* zold;
  const SolverState* s;
  long long N;
  double* partial;
  int gx;
};

__global__ __launch_bounds__(kBlock) void k_update_xr_g(const UpdateXrJob* __restrict__ jobs,
                                                        const int* __restrict__ start, int njobs) {
  const int j = group_job(start, njobs, (int)blockIdx.x);
  const UpdateXrJob& t = jobs[j];
  if (t.s->flag != FLAG_RUNNING) return;
  update_xr_body(t.x, t.r, t.p, t.q, t.zold, t.s, t.N, t.partial, (int)blockIdx.x - start[j], t.gx);
}

// p = z + beta p (beta = 0 on the first direction: p = z).
__global__ __launch_bounds__(kBlock) void k_update_p(double* __restrict__ p, const double* __restrict__ z,
                                                     const SolverState* __restrict__ s, int first, long long N) {
  if (!first && s->flag != FLAG_RUNNING) return;
  const double beta = first ? 0.0 : s->beta;
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (i < N) p[i] = first ? z[i] : fma(beta, p[i], z[i]);
}

struct UpdatePJob {
  double* p;
  const double* z;
  const SolverState* s;
  long long N;
};

template <bool FIRST>
__global__ __launch_bounds__(kBlock) void k_update_p_g(const UpdatePJob* __restrict__ jobs,
                                                       const int* __restrict__ start, int njobs) {
  const int j = group_job(start, njobs, (int)blockIdx.x);
  const UpdatePJob& t = jobs[j];
  if (!FIRST && t.s->flag != FLAG_RUNNING) return;
  const long long i = (long long)((int)blockIdx.x - start[j]) * kBlock + threadIdx.x;
  if (i < t.N) t.p[i] = FIRST ? t.z[i] : fma(t.s->beta, t.p[i], t.z[i]);
}

// flags[j] = the CG flag of problem j (one copy to the host per check)
__global__ void k_gather_flags(SolverState* const* __restrict__ states, int n, int* __restrict__ flags) {
  const int j = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (j < n) flags[j] = states[j]->flag;
}

// r = b - q and its squared norm (true residual).
__global__ __launch_bounds__(kBlock) void k_residual(const double* __restrict__ b, const double* __restrict__ q,
                                                     double* __restrict__ r, long long N, double* __restrict__ partial) {
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  double rr = 0.0;
  if (i < N) {
    const double ri = b[i] - q[i];
    r[i] = ri;
    rr = ri * ri;
  }
  const double t = block_sum(rr);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

void free_dev(void* p) {
  if (p) (void)hipFree(p);
}

unsigned vblocks(const igafd_ctx* c) { return (unsigned)((c->N + kBlock - 1) / kBlock); }

template <typename T>
igafd_status dev_upload(T** dst, const T* src, size_t count, hipStream_t st) {
  IGAFD_HIP_CHECK(device_malloc((void**)dst, sizeof(T) * (count ? count : 1)));
  if (count) IGAFD_HIP_CHECK(hipMemcpyAsync(*dst, src, sizeof(T) * count, hipMemcpyHostToDevice, st));
  return IGAFD_OK;
}

uint16_t to_bf16_host(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Device copies of a direction's element tables and the diagonals of M, K.
igafd_status upload_tables(const Dir1D& h, DevDir* d, hipStream_t st) {
  d->n = h.n;
  d->nel = h.nel;
  d->npad = fd_npad(h.n);
  igafd_status s;
  if ((s = dev_upload(&d->elem_first, h.elem_first.data(), h.elem_first.size(), st)) != IGAFD_OK) return s;
  std::vector<int> at((size_t)h.n + 2, -1);
  for (int e = 0; e < h.nel; ++e) at[h.elem_first[e]] = e;
  if ((s = dev_upload(&d->elem_at, at.data(), at.size(), st)) != IGAFD_OK) return s;
  if ((s = dev_upload(&d->qx, h.qx.data(), h.qx.size(), st)) != IGAFD_OK) return s;
  if ((s = dev_upload(&d->qw, h.qw.data(), h.qw.size(), st)) != IGAFD_OK) return s;
  if ((s = dev_upload(&d->val, h.val.data(), h.val.size(), st)) != IGAFD_OK) return s;
  if ((s = dev_upload(&d->der, h.der.data(), h.der.size(), st)) != IGAFD_OK) return s;
  const int n = h.n;
  std::vector<double> dm(n), dk(n);
  for (int i = 0; i < n; ++i) {
    dm[i] = h.M[(size_t)i * n + i];
    dk[i] = h.K[(size_t)i * n + i];
  }
  if ((s = dev_upload(&d->diagM, dm.data(), dm.size(), st)) != IGAFD_OK) return s;
  if ((s = dev_upload(&d->diagK, dk.data(), dk.size(), st)) != IGAFD_OK) return s;
  IGAFD_HIP_CHECK(hipStreamSynchronize(st));  // the host copies must outlive the asynchronous uploads
  return IGAFD_OK;
}

// Device copies of its eigenvalues, U^T and U in three precisions (zero padded
// to npad x npad).
igafd_status upload_eigen(const Dir1D& h, DevDir* d, hipStream_t st) {
  const int n = h.n, np = d->npad;
  igafd_status s;
  if ((s = dev_upload(&d->lam, h.lam.data(), h.lam.size(), st)) != IGAFD_OK) return s;
  std::vector<double> w64((size_t)np * np);
  std::vector<float> w32((size_t)np * np);
  std::vector<uint16_t> wbf((size_t)np * np);
  for (int which = 0; which < 2; ++which) {
    std::fill(w64.begin(), w64.end(), 0.0);
    for (int a = 0; a < n; ++a)
      for (int b = 0; b < n; ++b) w64[(size_t)a * np + b] = which == 0 ? h.U[(size_t)b * n + a] : h.U[(size_t)a * n + b];
    for (size_t k = 0; k < w64.size(); ++k) {
      w32[k] = (float)w64[k];
      wbf[k] = to_bf16_host((float)w64[k]);
    }
    if ((s = dev_upload(&d->W64[which], w64.data(), w64.size(), st)) != IGAFD_OK) return s;
    if ((s = dev_upload(&d->W32[which], w32.data(), w32.size(), st)) != IGAFD_OK) return s;
    if ((s = dev_upload(&d->Wbf[which], wbf.data(), wbf.size(), st)) != IGAFD_OK) return s;
    IGAFD_HIP_CHECK(hipStreamSynchronize(st));  // host staging vectors are reused
  }
  return IGAFD_OK;
}

// The eigendecompositions of the given directions: equal ones (same degree and
// knots) once, the others on a thread each.
igafd_status eigen_all(const std::vector<Dir1D*>& dirs) {
  std::vector<int> same(dirs.size());
  std::vector<igafd_status> st(dirs.size(), IGAFD_OK);
  std::vector<std::thread> th;
  for (size_t i = 0; i < dirs.size(); ++i) {
    same[i] = (int)i;
    for (size_t j = 0; j < i && same[i] == (int)i; ++j)
      if (dirs[j]->p == dirs[i]->p && dirs[j]->q == dirs[i]->q && dirs[j]->knots == dirs[i]->knots) same[i] = (int)j;
  }
  auto work = [&](size_t i) { return std::pow((double)dirs[i]->n, 3); };
  double all = 0.0;
  for (size_t i = 0; i < dirs.size(); ++i)
    if (same[i] == (int)i) all += work(i);
  auto run = [&](size_t i) {  // on a thread of its own: nothing may leave it
    try {
      st[i] = eigen_direction(dirs[i], eigen_threads(work(i) / all));
    } catch (const std::exception&) {
      st[i] = IGAFD_ERR_ALLOC;
    }
  };
  th.reserve(dirs.size());
  for (size_t i = 1; i < dirs.size(); ++i) {
    if (same[i] != (int)i) continue;
    try {
      th.emplace_back(run, i);
    } catch (const std::exception&) {  // no thread to be had
      run(i);
    }
  }
  run(0);
  for (std::thread& t : th) t.join();
  for (size_t i = 0; i < dirs.size(); ++i) {
    if (st[i] != IGAFD_OK) {
      set_error(st[i] == IGAFD_ERR_ALLOC ? "out of host memory" : "Cholesky of the 1D mass matrix failed");
      return st[i];
    }
    if (same[i] != (int)i) {
      dirs[i]->U = dirs[same[i]]->U;
      dirs[i]->lam = dirs[same[i]]->lam;
    }
  }
  return IGAFD_OK;
}

void free_dir(DevDir* d) {
  free_dev(d->elem_first);
  free_dev(d->elem_at);
  free_dev(d->qx);
  free_dev(d->qw);
  free_dev(d->val);
  free_dev(d->der);
  free_dev(d->lam);
  for (int w = 0; w < 2; ++w) {
    free_dev(d->W64[w]);
    free_dev(d->W32[w]);
    free_dev(d->Wbf[w]);
  }
  free_dev(d->diagM);
  free_dev(d->diagK);
  *d = DevDir{};
}

// the scratch allocation, cut into the given N-vectors (each 256-byte aligned)
igafd_status alloc_scratch(igafd_ctx* c, std::initializer_list<double**> vecs) {
  const long long nv = (c->N + 31) / 32 * 32;
  c->scratch_len = std::max((long long)vecs.size() * nv, load_scratch(c));
  const size_t bytes = sizeof(double) * (size_t)c->scratch_len;
  const igafd_status s = block_alloc((void**)&c->scratch, bytes);
  if (s != IGAFD_OK) return s;
  IGAFD_HIP_CHECK(hipMemsetAsync(c->scratch, 0, bytes, c->stream));
  double* p = c->scratch;
  for (double** v : vecs) {
    *v = p;
    p += nv;
  }
  return IGAFD_OK;
}

// Preconditioner-only context of one Schwarz subdomain (2D): the univariate
// eigendecompositions of its two knot vectors and the FD intermediates; no A.
igafd_status create_fd_sub(int p, const Dir1D& d1, const Dir1D& d2, hipStream_t st, igafd_ctx** out) {
  std::unique_ptr<igafd_ctx, void (*)(igafd_ctx*)> c(new igafd_ctx(), igafd_destroy);
  c->dim = 2;
  c->p = p;
  c->stream = st;
  IGAFD_HIP_CHECK(hipGetDevice(&c->device));
  c->N = 1;
  c->dir[0] = d1;
  c->dir[1] = d2;
  if (const char* e = std::getenv("IGAFD_FD_GEMM")) c->fd_gemm = std::atoi(e) != 0;
  igafd_status s;
  for (int l = 0; l < 2; ++l) {
    c->n[l] = c->dir[l].n;
    c->N *= c->n[l];
    if ((s = upload_tables(c->dir[l], &c->ddir[l], st)) != IGAFD_OK) return s;
    if ((s = upload_eigen(c->dir[l], &c->ddir[l], st)) != IGAFD_OK) return s;
  }
  if ((s = alloc_scratch(c.get(), {&c->fdbuf[0], &c->fdbuf[1]})) != IGAFD_OK) return s;
  *out = c.release();
  return IGAFD_OK;
}

bool no_A(const igafd_ctx* c, const char* what) {
  if (c->band) return false;
  set_error(std::string(what) + " needs A; this context holds only the preconditioner (igafd_setup_precond)");
  return true;
}

bool is_lshape(const igafd_ctx* c, const char* what) {
  if (c->hole < 0) return false;
  set_error(std::string(what) + " is not defined for the L-shaped multi-patch context");
  return true;
}

long long band_nnz(const igafd_ctx* c) {
  long long nnz = 1;
  for (int l = 0; l < c->dim; ++l) {
    long long cnt = 0;
    for (int i = 0; i < c->n[l]; ++i) {
      const int lo = std::max(0, i - c->p), hi = std::min(c->n[l] - 1, i + c->p);
      cnt += hi - lo + 1;
    }
    nnz *= cnt;
  }
  return nnz;
}

igafd_status parse_geometry(const igafd_problem* pr, GeomDesc* g) {
  std::memset(g, 0, sizeof(*g));
  g->dim = pr->dim;
  g->kind = pr->geom_kind;
  const double* gp = pr->geom_params;
  switch (pr->geom_kind) {
    case IGAFD_GEOM_IDENTITY:
    case IGAFD_GEOM_RING:
      break;
    case IGAFD_GEOM_WARPED: {
      if (!gp || pr->n_geom_params < 2) {
        set_error("warped geometry needs [a, K, c..., m...]");
        return IGAFD_ERR_ARG;
      }
      const int K = (int)gp[1];
      if (K < 0 || K > kMaxModes || pr->n_geom_params != 2 + 2 * K * pr->dim) {
        set_error("warped geometry: bad mode count or parameter length");
        return IGAFD_ERR_ARG;
      }
      g->amp = gp[0];
      g->nmodes = K;
      for (int k = 0; k < K; ++k)
        for (int l = 0; l < pr->dim; ++l) {
          g->c[k][l] = gp[2 + k * pr->dim + l];
          g->m[k][l] = gp[2 + K * pr->dim + k * pr->dim + l];
        }
      break;
    }
    default:
      set_error("unknown geometry kind");
      return IGAFD_ERR_ARG;
  }
  g->coef_kind = pr->coef_kind;
  switch (pr->coef_kind) {
    case IGAFD_COEF_ONE:
      break;
    case IGAFD_COEF_SINCOS:
      if (!pr->coef_params || pr->n_coef_params != 5) {
        set_error("sincos coefficient needs [a, f1, f2, phi1, phi2]");
        return IGAFD_ERR_ARG;
      }
      g->camp = pr->coef_params[0];
      g->f1 = pr->coef_params[1];
      g->f2 = pr->coef_params[2];
      g->phi1 = pr->coef_params[3];
      g->phi2 = pr->coef_params[4];
      break;
    default:
      set_error("unknown coefficient kind");
      return IGAFD_ERR_ARG;
  }
  return IGAFD_OK;
}

igafd_status alloc_workspace(igafd_ctx* c) {
  igafd_status s = alloc_scratch(c, {&c->r, &c->z, &c->zold, &c->q, &c->fdbuf[0], &c->fdbuf[1]});
  if (s != IGAFD_OK) return s;
  const size_t pb = sizeof(double) * (size_t)c->Ns;
  if ((s = block_alloc((void**)&c->pv_pad, pb)) != IGAFD_OK) return s;
  if ((s = block_alloc((void**)&c->xpad, pb)) != IGAFD_OK) return s;
  IGAFD_HIP_CHECK(hipMemsetAsync(c->pv_pad, 0, pb, c->stream));
  IGAFD_HIP_CHECK(hipMemsetAsync(c->xpad, 0, pb, c->stream));
  c->pv = c->pv_pad + c->halo;
  // partial sums: one (or two) per block of every reduction kernel, for any
  // kernel shape the autotuner may pick
  c->npartial = partial_capacity(c);
  IGAFD_HIP_CHECK(device_malloc((void**)&c->partial, sizeof(double) * 2 * (size_t)c->npartial));
  IGAFD_HIP_CHECK(device_malloc((void**)&c->state, sizeof(SolverState)));
  IGAFD_HIP_CHECK(hipHostMalloc((void**)&c->hstate, sizeof(SolverState), hipHostMallocDefault));
  IGAFD_HIP_CHECK(device_malloc((void**)&c->dflag, sizeof(int)));
  IGAFD_HIP_CHECK(hipEventCreate(&c->ev0));
  IGAFD_HIP_CHECK(hipEventCreate(&c->ev1));
  // residual history for the default iteration budget (maxit 2000 + the start)
  c->hist_alloc = kHistDefault;
  IGAFD_HIP_CHECK(device_malloc((void**)&c->hist, sizeof(double) * c->hist_alloc));
  return IGAFD_OK;
}

// Phase timers of a timed solve.  mark(c, ph) records an event that opens a
// segment of phase ph (PH_NONE closes the previous one without opening a new
// segment); harvest(c), called once the stream has drained, adds the elapsed
// time of every recorded segment to its phase.
enum { PH_NONE = -1, PH_SPMV = 0, PH_FD = 1, PH_VEC = 2 };

igafd_status mark(igafd_ctx* c, int ph) {
  if (!c->timing) return IGAFD_OK;
  if (c->tused == (int)c->tev.size()) {
    hipEvent_t e = nullptr;
    IGAFD_HIP_CHECK(hipEventCreate(&e));
    c->tev.push_back(e);
    c->tphase.push_back(PH_NONE);
  }
  IGAFD_HIP_CHECK(hipEventRecord(c->tev[c->tused], c->stream));
  c->tphase[c->tused] = ph;
  c->tused += 1;
  return IGAFD_OK;
}

igafd_status harvest(igafd_ctx* c) {
  if (!c->timing) return IGAFD_OK;
  for (int k = 0; k + 1 < c->tused; ++k) {
    if (c->tphase[k] == PH_NONE) continue;
    float ms = 0.f;
    IGAFD_HIP_CHECK(hipEventElapsedTime(&ms, c->tev[k], c->tev[k + 1]));
    c->tacc[c->tphase[k]] += ms;
  }
  c->tused = 0;
  return IGAFD_OK;
}

// every reduction writes at most npartial (x 2) block partials
igafd_status check_partials(const igafd_ctx* c, long long blocks) {
  if (blocks > c->npartial) {
    set_error("internal: reduction grid larger than the partial-sum buffer");
    return IGAFD_ERR_ARG;
  }
  return IGAFD_OK;
}

igafd_status reduce(igafd_ctx* c, int count, int two, int which, double* hist) {
  if (count > c->npartial) {
    set_error("internal: reduction count larger than the partial-sum buffer");
    return IGAFD_ERR_ARG;
  }
  hipLaunchKernelGGL(k_reduce, dim3(1), dim3(kReduceBlock), 0, c->stream, c->partial, count, two, which, c->state,
                     hist);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status read_state(igafd_ctx* c) {
  if (mark(c, PH_NONE) != IGAFD_OK) return IGAFD_ERR_HIP;
  IGAFD_HIP_CHECK(hipMemcpyAsync(c->hstate, c->state, sizeof(SolverState), hipMemcpyDeviceToHost, c->stream));
  IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
  return harvest(c);
}

#define IGAFD_TRY(x)                          \
  do {                                        \
    igafd_status st_ = (x);                   \
    if (st_ != IGAFD_OK) return st_;          \
  } while (0)

// z = M r with M = P^-1 or S P^-1 S; (r, z) partials; then rho or beta.
igafd_status precond_step(igafd_ctx* c, int prec, const double* S, double* z, int which, const int* flag) {
  IGAFD_TRY(fd_apply(c, prec, c->r, z, S, c->partial, flag));
  return reduce(c, fd_dot_blocks(c, prec), 0, which, nullptr);
}

// (Re)start: r holds the residual; z = M r, rho = (r, z), p = z.
igafd_status start_directions(igafd_ctx* c, int prec, const double* S, double*& z, double*& zold) {
  IGAFD_TRY(mark(c, PH_FD));
  IGAFD_TRY(fd_apply(c, prec, c->r, z, S, c->partial, nullptr));
  IGAFD_TRY(reduce(c, fd_dot_blocks(c, prec), 0, RED_RHO0, nullptr));
  IGAFD_TRY(mark(c, PH_VEC));
  hipLaunchKernelGGL(k_update_p, dim3(vblocks(c)), dim3(kBlock), 0, c->stream, c->pv, z, c->state, 1, c->N);
  IGAFD_HIP_CHECK(hipGetLastError());
  (void)zold;
  return IGAFD_OK;
}

// One CG iteration, enqueued without any host synchronisation (also used
// under graph capture).  z / zold swap roles every iteration.
igafd_status enqueue_iteration(igafd_ctx* c, double* x, int prec, const double* S, int flexible, double*& z,
                               double*& zold, double* hist) {
  const unsigned vb = vblocks(c);
  const int* flag = &c->state->flag;
  IGAFD_TRY(check_partials(c, (long long)vb));
  // q = A p, (p, q)
  IGAFD_TRY(mark(c, PH_SPMV));
  IGAFD_TRY(spmv(c, c->pv, c->q, c->partial, flag));
  IGAFD_TRY(reduce(c, spmv_blocks(c), 0, RED_PQ, hist));
  // x += alpha p, r -= alpha q, (r, r) [, (r, z_old)]
  IGAFD_TRY(mark(c, PH_VEC));
  hipLaunchKernelGGL(k_update_xr, dim3(vb), dim3(kBlock), 0, c->stream, x, c->r, c->pv, c->q, flexible ? z : nullptr,
                     c->state, c->N, c->partial);
  IGAFD_HIP_CHECK(hipGetLastError());
  IGAFD_TRY(reduce(c, (int)vb, flexible, RED_RR, hist));
  // z = M r, (r, z) -> beta; the previous z stays as z_old for the flexible form
  std::swap(z, zold);
  IGAFD_TRY(mark(c, PH_FD));
  IGAFD_TRY(precond_step(c, prec, S, z, RED_RZ, flag));
  IGAFD_TRY(mark(c, PH_VEC));
  hipLaunchKernelGGL(k_update_p, dim3(vb), dim3(kBlock), 0, c->stream, c->pv, z, c->state, 0, c->N);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status check_opts(const igafd_ctx* c, const igafd_solve_opts* o) {
  if (o->precision != IGAFD_FP64 && !o->flexible) {
    set_error("FP32/BF16 preconditioner applies need the flexible CG form");
    return IGAFD_ERR_ARG;
  }
  if (o->precision < IGAFD_FP64 || o->precision > IGAFD_BF16X3) {
    set_error("unknown precision");
    return IGAFD_ERR_ARG;
  }
  if (!(o->rtol > 0.0)) {
    set_error("rtol must be positive");
    return IGAFD_ERR_ARG;
  }
  if (o->use_scaling < 0 || o->use_scaling > 2) {
    set_error("use_scaling must be 0, 1 or 2");
    return IGAFD_ERR_ARG;
  }
  if (c->adi && (o->precision != IGAFD_FP64 || o->use_scaling == 1)) {
    set_error("the ADI preconditioner runs in FP64 and without scaling");
    return IGAFD_ERR_ARG;
  }
  if (o->use_scaling == 1 && !c->scaling_set) {
    set_error("use_scaling requested but no scaling set");
    return IGAFD_ERR_ARG;
  }
  return IGAFD_OK;
}

// Scaling gate (Sec. 3, Prop. 1): the spectrum of P^-1 A lies in
// [qmin, qmax], the extreme eigenvalues of Q over the Gauss points.  A diagonal
// scaling S P^-1 S can at best remove the variation of Q's magnitude over the
// domain, not the anisotropy of Q at a point, so no such scaling brings the
// corresponding bound below qloc = max_x lambda_max(Q(x)) / lambda_min(Q(x)).
// The gate passes when the bound could shrink by at least `gain`:
// (qmax / qmin) / qloc >= gain.
igafd_status gate_impl(igafd_ctx* c, double gain, int* use, double* kappa_q, double* kappa_loc) {
  double lo = 0.0, hi = 0.0, loc = 0.0;
  IGAFD_TRY(spectral_bounds(c, &lo, &hi, &loc));
  const double kq = hi / lo;
  if (kappa_q) *kappa_q = kq;
  if (kappa_loc) *kappa_loc = loc;
  if (use) *use = (kq >= gain * loc) ? 1 : 0;
  return IGAFD_OK;
}

constexpr double kGateGain = 2.0;  // default gain of use_scaling = 2

igafd_status solve_impl(igafd_ctx* c, const double* b, double* x, const igafd_solve_opts* o, igafd_solve_info* info) {
  const int maxit = o->maxit > 0 ? o->maxit : 2000;
  const int chunk = o->check_every > 0 ? o->check_every : 4;
  const int prec = o->precision;
  const int flexible = o->flexible ? 1 : 0;
  IGAFD_TRY(check_opts(c, o));
  double kappa_bound = 0.0;
  bool scaled = o->use_scaling == 1;
  if (o->use_scaling == 2 && c->hole < 0) {
    int pass = 0;
    IGAFD_TRY(gate_impl(c, kGateGain, &pass, &kappa_bound, nullptr));
    scaled = pass && c->scaling_set && !c->adi;
  }
  const double* S = scaled ? c->scaling : nullptr;
  // residual history: the context's device buffer, grown once for maxit > 2000
  double* hist = nullptr;
  const int hcap = o->history ? maxit + 1 : 0;
  if (hcap > c->hist_alloc) {
    IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
    if (c->hist) IGAFD_HIP_CHECK(hipFree(c->hist));
    c->hist = nullptr;
    c->hist_alloc = 0;
    IGAFD_HIP_CHECK(device_malloc((void**)&c->hist, sizeof(double) * hcap));
    c->hist_alloc = hcap;
  }
  if (hcap) hist = c->hist;
  const unsigned vb = vblocks(c);
  c->timing = o->timers != 0;
  c->tused = 0;
  c->tacc[0] = c->tacc[1] = c->tacc[2] = 0.0;
  // the timers must be off again on every return path (the batched solve
  // captures the same enqueue code into graphs)
  struct TimingOff {
    igafd_ctx* c;
    ~TimingOff() { c->timing = false; }
  } timing_off{c};
  IGAFD_HIP_CHECK(hipEventRecord(c->ev0, c->stream));

  SolverState init{};
  init.tol2 = o->rtol * o->rtol;
  init.maxit = maxit;
  init.flexible = flexible;
  init.hist_cap = hcap;
  *c->hstate = init;
  IGAFD_TRY(mark(c, PH_VEC));
  IGAFD_HIP_CHECK(hipMemcpyAsync(c->state, c->hstate, sizeof(SolverState), hipMemcpyHostToDevice, c->stream));
  const double* y = nullptr;
  if (o->use_x0) {
    IGAFD_TRY(mark(c, PH_SPMV));
    IGAFD_TRY(spmv_unpadded(c, x, c->q, nullptr, nullptr));
    IGAFD_TRY(mark(c, PH_VEC));
    y = c->q;
  }
  IGAFD_TRY(check_partials(c, (long long)vb));
  hipLaunchKernelGGL(k_init, dim3(vb), dim3(kBlock), 0, c->stream, b, y, c->r, x, o->use_x0 ? 1 : 0, c->N, c->partial);
  IGAFD_HIP_CHECK(hipGetLastError());
  IGAFD_TRY(reduce(c, (int)vb, 1, RED_BB_RR, hist));
  IGAFD_TRY(read_state(c));
  const double bb = c->hstate->bb;

  double* z = c->z;
  double* zold = c->zold;
  int restarts = 0, fell_back = 0;
  double true_rel = 0.0;
  int status = IGAFD_OK;
  while (true) {
    if (c->hstate->flag == FLAG_RUNNING) {
      IGAFD_TRY(start_directions(c, prec, S, z, zold));
      while (true) {
        for (int k = 0; k < chunk; ++k) IGAFD_TRY(enqueue_iteration(c, x, prec, S, flexible, z, zold, hist));
        IGAFD_TRY(read_state(c));
        if (c->hstate->flag != FLAG_RUNNING) break;
      }
    }
    // true residual in FP64
    IGAFD_TRY(mark(c, PH_SPMV));
    IGAFD_TRY(spmv_unpadded(c, x, c->q, nullptr, nullptr));
    IGAFD_TRY(mark(c, PH_VEC));
    hipLaunchKernelGGL(k_residual, dim3(vb), dim3(kBlock), 0, c->stream, b, c->q, c->r, c->N, c->partial);
    IGAFD_HIP_CHECK(hipGetLastError());
    IGAFD_TRY(reduce(c, (int)vb, 0, RED_TRUE, nullptr));
    IGAFD_TRY(read_state(c));
    const SolverState hs = *c->hstate;
    true_rel = bb > 0.0 ? std::sqrt(hs.rrtrue / bb) : 0.0;
    if (true_rel <= o->rtol && hs.flag != FLAG_BREAKDOWN) {
      status = IGAFD_OK;
      break;
    }
    const bool stuck = hs.flag == FLAG_BREAKDOWN || hs.iters >= c->hstate->maxit || restarts >= 3;
    if (stuck && S && std::isfinite(true_rel)) {
      // the scaled preconditioner stagnated or broke down: continue from the
      // current iterate with plain P and a fresh iteration budget
      S = nullptr;
      fell_back = 1;
      c->hstate->maxit = hs.iters + maxit;
      IGAFD_HIP_CHECK(hipMemcpyAsync(&c->state->maxit, &c->hstate->maxit, sizeof(int), hipMemcpyHostToDevice,
                                     c->stream));
    } else if (hs.flag == FLAG_BREAKDOWN) {
      status = IGAFD_ERR_BREAKDOWN;
      break;
    } else if (stuck) {
      status = IGAFD_NOT_CONVERGED;
      break;
    }
    // restart from the true residual (held in r)
    ++restarts;
    c->hstate->flag = FLAG_RUNNING;
    IGAFD_HIP_CHECK(hipMemcpyAsync(&c->state->flag, &c->hstate->flag, sizeof(int), hipMemcpyHostToDevice, c->stream));
  }
  IGAFD_HIP_CHECK(hipEventRecord(c->ev1, c->stream));
  IGAFD_TRY(read_state(c));
  const SolverState hs = *c->hstate;
  float ms = 0.f;
  IGAFD_HIP_CHECK(hipEventSynchronize(c->ev1));
  IGAFD_HIP_CHECK(hipEventElapsedTime(&ms, c->ev0, c->ev1));
  int nh = 0;
  if (hist) {
    nh = std::min(hs.iters + 1, hcap);
    IGAFD_HIP_CHECK(hipMemcpyAsync(o->history, hist, sizeof(double) * nh, hipMemcpyDeviceToHost, c->stream));
    IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
  }
  if (info) {
    info->iters = hs.iters;
    info->restarts = restarts;
    info->true_relres = true_rel;
    info->status = status;
    info->t_solve_ms = ms;
    info->relres = bb > 0.0 ? std::sqrt(hs.rr / bb) : 0.0;
    info->fallback = fell_back;
    info->history_len = nh;
    info->t_setup_ms = c->t_setup_ms;
    info->t_spmv_ms = c->tacc[PH_SPMV];
    info->t_fd_ms = c->tacc[PH_FD];
    info->t_vec_ms = c->tacc[PH_VEC];
    info->scaled = scaled ? 1 : 0;
    info->kappa_bound = kappa_bound;
  }
  if (status == IGAFD_ERR_BREAKDOWN) set_error("CG breakdown: p^T A p <= 0 or not finite");
  return (igafd_status)status;
}

}  // namespace

size_t GroupArena::push(const void* p, size_t bytes) {
  const size_t off = (host.size() + 63) / 64 * 64;
  host.resize(off + bytes);
  if (bytes) std::memcpy(host.data() + off, p, bytes);
  return off;
}

igafd_status GroupArena::upload(hipStream_t st) {
  if (host.empty()) return IGAFD_OK;
  if (!dev || cap < host.size()) {
    IGAFD_HIP_CHECK(hipStreamSynchronize(st));  // launches reading the old tables are done
    if (dev) IGAFD_HIP_CHECK(hipFree(dev));
    dev = nullptr;
    cap = 0;
    IGAFD_HIP_CHECK(device_malloc((void**)&dev, host.size()));
    cap = host.size();
  }
  IGAFD_HIP_CHECK(hipMemcpyAsync(dev, host.data(), host.size(), hipMemcpyHostToDevice, st));
  IGAFD_HIP_CHECK(hipStreamSynchronize(st));
  return IGAFD_OK;
}

void GroupArena::release() {
  if (dev) (void)hipFree(dev);
  dev = nullptr;
  cap = 0;
  host.clear();
}

namespace {

// The launches of one CG iteration (the steps of enqueue_iteration) for the
// problems `run`, each step one grouped launch over all of them (the tiled A
// product and the slice passes: one per kernel shape).  steps[0]: z[i] holds
// the current z (the flexible form's z_old of this iteration), the new z goes
// to zold[i]; steps[1]: the roles swapped (the next iteration).  *flags_off:
// the table of state pointers for k_gather_flags.
igafd_status build_grouped(GroupArena& a, std::vector<GroupStep> (&steps)[2], size_t* flags_off,
                           const std::vector<int>& run, igafd_ctx* const* cs, double* const* xs, int prec,
                           int flexible, const std::vector<const double*>& Sp, const std::vector<double*>& z,
                           const std::vector<double*>& zold) {
  a.host.clear();
  steps[0].clear();
  steps[1].clear();
  const int n = (int)run.size();
  std::vector<igafd_ctx*> cc;
  std::vector<const double*> pv, rv, S;
  std::vector<double*> q, part;
  std::vector<SolverState*> states;
  for (int i : run) {
    igafd_ctx* c = cs[i];
    IGAFD_TRY(check_partials(c, (long long)vblocks(c)));
    cc.push_back(c);
    pv.push_back(c->pv);
    rv.push_back(c->r);
    S.push_back(Sp[i]);
    q.push_back(c->q);
    part.push_back(c->partial);
    states.push_back(c->state);
  }
  *flags_off = a.push(states.data(), sizeof(SolverState*) * states.size());
  auto red_table = [&](int which, int two) -> long long {
    std::vector<ReduceJob> jobs;
    for (igafd_ctx* c : cc) {
      const int count = which == RED_PQ ? spmv_blocks(c) : which == RED_RR ? (int)vblocks(c) : fd_dot_blocks(c, prec);
      if (count > c->npartial) return -1;
      jobs.push_back(ReduceJob{c->partial, count, two, c->state});
    }
    return (long long)a.push(jobs.data(), sizeof(ReduceJob) * jobs.size());
  };
  const long long red_pq = red_table(RED_PQ, 0), red_rr = red_table(RED_RR, flexible), red_rz = red_table(RED_RZ, 0);
  if (red_pq < 0 || red_rr < 0 || red_rz < 0) {
    set_error("internal: reduction count larger than the partial-sum buffer");
    return IGAFD_ERR_ARG;
  }
  auto reduce_step = [&a, n](long long off, int which) -> GroupStep {
    return [&a, n, off, which](hipStream_t st) -> igafd_status {
      hipLaunchKernelGGL(k_reduce_g, dim3((unsigned)n), dim3(kReduceBlock), 0, st, a.at<ReduceJob>((size_t)off),
                         which);
      IGAFD_HIP_CHECK(hipGetLastError());
      return IGAFD_OK;
    };
  };
  for (int par = 0; par < 2; ++par) {
    std::vector<double*> za, zb;
    for (int i : run) {
      za.push_back(par ? zold[i] : z[i]);
      zb.push_back(par ? z[i] : zold[i]);
    }
    std::vector<GroupStep>& st = steps[par];
    // q = A p, (p, q)
    IGAFD_TRY(spmv_grouped(a, st, cc, pv, q, part));
    st.push_back(reduce_step(red_pq, RED_PQ));
    // x += alpha p, r -= alpha q, (r, r) [, (r, z_old)]
    {
      std::vector<UpdateXrJob> jobs;
      std::vector<int> start(1, 0);
      for (int k = 0; k < n; ++k) {
        igafd_ctx* c = cc[k];
        const int vb = (int)vblocks(c);
        jobs.push_back(UpdateXrJob{xs[run[k]], c->r, c->pv, c->q, flexible ? za[k] : nullptr, c->state, c->N,
                                   c->partial, vb});
        start.push_back(start.back() + vb);
      }
      const size_t oj = a.push(jobs.data(), sizeof(UpdateXrJob) * jobs.size());
      const size_t os = a.push(start.data(), sizeof(int) * start.size());
      const int blocks = start.back();
      st.push_back([&a, oj, os, n, blocks](hipStream_t s0) -> igafd_status {
        hipLaunchKernelGGL(k_update_xr_g, dim3((unsigned)blocks), dim3(kBlock), 0, s0, a.at<UpdateXrJob>(oj),
                           a.at<int>(os), n);
        IGAFD_HIP_CHECK(hipGetLastError());
        return IGAFD_OK;
      });
    }
    st.push_back(reduce_step(red_rr, RED_RR));
    // z = M r, (r, z) -> beta
    std::vector<double*> zbo(zb.begin(), zb.end());
    IGAFD_TRY(fd_grouped(a, st, cc, prec, rv, zbo, S, part));
    st.push_back(reduce_step(red_rz, RED_RZ));
    // p = z + beta p
    {
      std::vector<UpdatePJob> jobs;
      std::vector<int> start(1, 0);
      for (int k = 0; k < n; ++k) {
        igafd_ctx* c = cc[k];
        jobs.push_back(UpdatePJob{c->pv, zb[k], c->state, c->N});
        start.push_back(start.back() + (int)vblocks(c));
      }
      const size_t oj = a.push(jobs.data(), sizeof(UpdatePJob) * jobs.size());
      const size_t os = a.push(start.data(), sizeof(int) * start.size());
      const int blocks = start.back();
      st.push_back([&a, oj, os, n, blocks](hipStream_t s0) -> igafd_status {
        hipLaunchKernelGGL(k_update_p_g<false>, dim3((unsigned)blocks), dim3(kBlock), 0, s0, a.at<UpdatePJob>(oj),
                           a.at<int>(os), n);
        IGAFD_HIP_CHECK(hipGetLastError());
        return IGAFD_OK;
      });
    }
  }
  return IGAFD_OK;
}

// Grouped phases of a batched solve outside the iteration loop, for the
// problems `ids` (each one launch per step, tables in `a`):
// init: r = b, x = 0, then ||b||^2, ||r||^2 and the stop test (RED_BB_RR);
// *flags_off: the table of state pointers for k_gather_flags.
igafd_status build_grouped_init(GroupArena& a, std::vector<GroupStep>& steps, size_t* flags_off,
                                const std::vector<int>& ids, igafd_ctx* const* cs, const double* const* bs,
                                double* const* xs) {
  a.host.clear();
  steps.clear();
  const int n = (int)ids.size();
  std::vector<InitJob> jobs;
  std::vector<ReduceJob> red;
  std::vector<SolverState*> states;
  std::vector<int> start(1, 0);
  for (int i : ids) {
    igafd_ctx* c = cs[i];
    const int vb = (int)vblocks(c);
    IGAFD_TRY(check_partials(c, vb));  // two sums of vb partials: the buffer holds 2 npartial
    jobs.push_back(InitJob{bs[i], nullptr, c->r, xs[i], c->N, c->partial, vb});
    red.push_back(ReduceJob{c->partial, vb, 1, c->state});
    states.push_back(c->state);
    start.push_back(start.back() + vb);
  }
  *flags_off = a.push(states.data(), sizeof(SolverState*) * states.size());
  const size_t oj = a.push(jobs.data(), sizeof(InitJob) * jobs.size());
  const size_t os = a.push(start.data(), sizeof(int) * start.size());
  const size_t orr = a.push(red.data(), sizeof(ReduceJob) * red.size());
  const int blocks = start.back();
  steps.push_back([&a, oj, os, orr, n, blocks](hipStream_t st) -> igafd_status {
    hipLaunchKernelGGL(k_init_g, dim3((unsigned)blocks), dim3(kBlock), 0, st, a.at<InitJob>(oj), a.at<int>(os), n);
    IGAFD_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_reduce_g, dim3((unsigned)n), dim3(kReduceBlock), 0, st, a.at<ReduceJob>(orr), (int)RED_BB_RR);
    IGAFD_HIP_CHECK(hipGetLastError());
    return IGAFD_OK;
  });
  return IGAFD_OK;
}

// first directions of the running problems: z = M r, rho = (r, z), p = z
igafd_status build_grouped_start(GroupArena& a, std::vector<GroupStep>& steps, const std::vector<int>& run,
                                 igafd_ctx* const* cs, int prec, const std::vector<const double*>& Sp,
                                 const std::vector<double*>& z) {
  a.host.clear();
  steps.clear();
  const int n = (int)run.size();
  std::vector<igafd_ctx*> cc;
  std::vector<const double*> rv, S;
  std::vector<double*> zz, part;
  std::vector<ReduceJob> red;
  std::vector<UpdatePJob> pj;
  std::vector<int> start(1, 0);
  for (int i : run) {
    igafd_ctx* c = cs[i];
    const int cnt = fd_dot_blocks(c, prec);
    IGAFD_TRY(check_partials(c, cnt));
    cc.push_back(c);
    rv.push_back(c->r);
    S.push_back(Sp[i]);
    zz.push_back(z[i]);
    part.push_back(c->partial);
    red.push_back(ReduceJob{c->partial, cnt, 0, c->state});
    pj.push_back(UpdatePJob{c->pv, z[i], c->state, c->N});
    start.push_back(start.back() + (int)vblocks(c));
  }
  IGAFD_TRY(fd_grouped(a, steps, cc, prec, rv, zz, S, part));
  const size_t orr = a.push(red.data(), sizeof(ReduceJob) * red.size());
  const size_t oj = a.push(pj.data(), sizeof(UpdatePJob) * pj.size());
  const size_t os = a.push(start.data(), sizeof(int) * start.size());
  const int blocks = start.back();
  steps.push_back([&a, orr, oj, os, n, blocks](hipStream_t st) -> igafd_status {
    hipLaunchKernelGGL(k_reduce_g, dim3((unsigned)n), dim3(kReduceBlock), 0, st, a.at<ReduceJob>(orr), (int)RED_RHO0);
    IGAFD_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_update_p_g<true>, dim3((unsigned)blocks), dim3(kBlock), 0, st, a.at<UpdatePJob>(oj),
                       a.at<int>(os), n);
    IGAFD_HIP_CHECK(hipGetLastError());
    return IGAFD_OK;
  });
  return IGAFD_OK;
}

// FP64 true residuals: x into the zero-halo buffer, q = A x (every problem,
// stopped or not), r = b - q, ||r||^2 (RED_TRUE)
igafd_status build_grouped_residual(GroupArena& a, std::vector<GroupStep>& steps, const std::vector<int>& ids,
                                    igafd_ctx* const* cs, const double* const* bs, double* const* xs) {
  a.host.clear();
  steps.clear();
  const int n = (int)ids.size();
  std::vector<igafd_ctx*> cc;
  std::vector<const double*> xp;
  std::vector<double*> q, nopart(n, nullptr);
  std::vector<CopyJob> cj;
  std::vector<InitJob> rj;
  std::vector<ReduceJob> red;
  std::vector<int> start(1, 0);
  for (int i : ids) {
    igafd_ctx* c = cs[i];
    const int vb = (int)vblocks(c);
    IGAFD_TRY(check_partials(c, vb));
    cc.push_back(c);
    xp.push_back(c->xpad + c->halo);
    q.push_back(c->q);
    cj.push_back(CopyJob{xs[i], c->xpad + c->halo, c->N});
    rj.push_back(InitJob{bs[i], c->q, c->r, nullptr, c->N, c->partial, vb});
    red.push_back(ReduceJob{c->partial, vb, 0, c->state});
    start.push_back(start.back() + vb);
  }
  const size_t oc = a.push(cj.data(), sizeof(CopyJob) * cj.size());
  const size_t os = a.push(start.data(), sizeof(int) * start.size());
  const int blocks = start.back();
  steps.push_back([&a, oc, os, n, blocks](hipStream_t st) -> igafd_status {
    hipLaunchKernelGGL(k_copy_g, dim3((unsigned)blocks), dim3(kBlock), 0, st, a.at<CopyJob>(oc), a.at<int>(os), n);
    IGAFD_HIP_CHECK(hipGetLastError());
    return IGAFD_OK;
  });
  IGAFD_TRY(spmv_grouped(a, steps, cc, xp, q, nopart, false));
  const size_t orj = a.push(rj.data(), sizeof(InitJob) * rj.size());
  const size_t orr = a.push(red.data(), sizeof(ReduceJob) * red.size());
  steps.push_back([&a, orj, orr, os, n, blocks](hipStream_t st) -> igafd_status {
    hipLaunchKernelGGL(k_init_g, dim3((unsigned)blocks), dim3(kBlock), 0, st, a.at<InitJob>(orj), a.at<int>(os), n);
    IGAFD_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_reduce_g, dim3((unsigned)n), dim3(kReduceBlock), 0, st, a.at<ReduceJob>(orr), (int)RED_TRUE);
    IGAFD_HIP_CHECK(hipGetLastError());
    return IGAFD_OK;
  });
  return IGAFD_OK;
}

bool batch_groupable(igafd_ctx* const* cs, int count, int prec) {
  if (const char* e = std::getenv("IGAFD_BATCH_GROUPED"))
    if (std::atoi(e) == 0) return false;
  for (int i = 0; i < count; ++i)
    if (!spmv_groupable(cs[i]) || !fd_groupable(cs[i], prec)) return false;
  return true;
}

// Several independent problems solved together.  When every problem is 3D
// with the fused FD passes, each step of a CG iteration is one grouped launch
// over all running problems (per kernel shape for the A product and the slice
// passes), from job tables built on the host: a chunk of iterations is
// captured once into a HIP graph on one stream and replayed.  Otherwise each
// context is bound to one stream of a small pool and the chunk is captured
// with fork/join over the pool.  Either way the graph is rebuilt when the
// running set shrinks enough, every kernel of a converged problem is a no-op
// (device stop flag), the per-problem arithmetic is that of a single solve
// (bitwise the same iterates), and problems that fail the FP64 true-residual
// check continue alone.
igafd_status solve_batched_impl(igafd_ctx* const* cs, int count, const double* const* bs, double* const* xs,
                                const igafd_solve_opts* o, igafd_solve_info* infos, double* wall_ms) {
  for (int i = 0; i < count; ++i) {
    if (!cs[i] || !bs[i] || !xs[i] || bs[i] == xs[i]) {
      set_error("batched solve needs a context and distinct b, u for every problem");
      return IGAFD_ERR_ARG;
    }
    IGAFD_TRY(check_opts(cs[i], o));
  }
  const int maxit = o->maxit > 0 ? o->maxit : 2000;
  int chunk = o->check_every > 0 ? o->check_every : 4;
  chunk += chunk & 1;  // even: the z / z_old roles return to the captured ones
  // preconditioner of each problem: S P^-1 S when asked for, or when the
  // Prop. 1 gate passes (use_scaling = 2); the gate runs on the caller's stream
  std::vector<const double*> Sp(count, nullptr);
  for (int i = 0; i < count; ++i) {
    bool use = o->use_scaling == 1;
    if (o->use_scaling == 2 && cs[i]->scaling_set) {
      int pass = 0;
      IGAFD_TRY(gate_impl(cs[i], kGateGain, &pass, nullptr, nullptr));
      use = pass != 0;
    }
    Sp[i] = use ? cs[i]->scaling : nullptr;
  }
  // every problem 3D with the fused FD passes: each step of an iteration one
  // grouped launch over all running problems; otherwise a pool of streams,
  // one problem's launches after another's
  const bool grouped = batch_groupable(cs, count, o->precision);
  int nst = 8;
  if (const char* e = std::getenv("IGAFD_BATCH_STREAMS")) nst = std::max(1, std::min(32, std::atoi(e)));
  nst = grouped ? 1 : std::min(nst, count);
  // streams by longest-processing-time first: problems in decreasing order of
  // the bytes their A band moves per iteration, each to the least loaded stream
  std::vector<int> slot(count, 0);
  {
    std::vector<int> order(count);
    for (int i = 0; i < count; ++i) order[i] = i;
    auto work = [&](int i) { return (double)cs[i]->H * (double)cs[i]->Ns + 8.0 * (double)cs[i]->N; };
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return work(a) > work(b); });
    std::vector<double> load(nst, 0.0);
    for (int i : order) {
      const int k = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      slot[i] = k;
      load[k] += work(i);
    }
  }
  std::vector<hipStream_t> pool(nst, nullptr), saved(count);
  std::vector<hipEvent_t> join(nst, nullptr);
  hipEvent_t fork = nullptr, t0 = nullptr, t1 = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  GroupArena arena;       // job tables of the grouped launches
  int* dflags = nullptr;  // the captured problems' CG flags, gathered per check
  igafd_status st = IGAFD_OK;
  std::vector<double*> z(count), zold(count);
  std::vector<char> running(count, 0);
  bool bound = false;  // the contexts are bound to the pool streams
  auto cleanup = [&]() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    for (hipStream_t q : pool)
      if (q) (void)hipStreamSynchronize(q);
    arena.release();
    if (dflags) (void)hipFree(dflags);
    // the callers' streams continue after everything the pool ran
    for (int k = 0; k < nst; ++k)
      if (pool[k] && join[k] && hipEventRecord(join[k], pool[k]) == hipSuccess)
        for (int i = 0; i < count; ++i)
          if (bound) (void)hipStreamWaitEvent(saved[i], join[k], 0);
    for (int k = 0; k < nst; ++k) {
      if (pool[k]) (void)hipStreamSynchronize(pool[k]);
    }
    if (bound)
      for (int i = 0; i < count; ++i) cs[i]->stream = saved[i];
    for (int k = 0; k < nst; ++k) {
      if (join[k]) (void)hipEventDestroy(join[k]);
      if (pool[k]) (void)hipStreamDestroy(pool[k]);
    }
    if (fork) (void)hipEventDestroy(fork);
    if (t0) (void)hipEventDestroy(t0);
    if (t1) (void)hipEventDestroy(t1);
  };
#define IGAFD_BT(x)              \
  do {                           \
    if ((st = (x)) != IGAFD_OK) {\
      cleanup();                 \
      return st;                 \
    }                            \
  } while (0)
#define IGAFD_BH(x)                                                              \
  do {                                                                           \
    hipError_t e_ = (x);                                                         \
    if (e_ != hipSuccess) {                                                      \
      set_error(std::string(#x) + ": " + hipGetErrorString(e_));                 \
      cleanup();                                                                 \
      return IGAFD_ERR_HIP;                                                      \
    }                                                                            \
  } while (0)
  for (int i = 0; i < count; ++i) saved[i] = cs[i]->stream;
  for (int k = 0; k < nst; ++k) {
    IGAFD_BH(hipStreamCreateWithFlags(&pool[k], hipStreamNonBlocking));
    IGAFD_BH(hipEventCreateWithFlags(&join[k], hipEventDisableTiming));
  }
  IGAFD_BH(hipEventCreateWithFlags(&fork, hipEventDisableTiming));
  IGAFD_BH(hipEventCreate(&t0));
  IGAFD_BH(hipEventCreate(&t1));
  // every pool stream first waits for the work already queued on the
  // streams of the contexts it takes over (uploads, load vectors, scalings)
  for (int i = 0; i < count; ++i) {
    IGAFD_BH(hipEventRecord(fork, saved[i]));
    IGAFD_BH(hipStreamWaitEvent(pool[slot[i]], fork, 0));
  }
  for (int i = 0; i < count; ++i) cs[i]->stream = pool[slot[i]];
  bound = true;
  auto sync_all = [&]() -> igafd_status {
    for (int k = 0; k < nst; ++k) IGAFD_HIP_CHECK(hipStreamSynchronize(pool[k]));
    return IGAFD_OK;
  };
  IGAFD_BH(hipEventRecord(t0, pool[0]));
  for (int k = 1; k < nst; ++k) IGAFD_BH(hipStreamWaitEvent(pool[k], t0, 0));
  // init: r = b, x = 0, ||b||, ||r||; then the first directions
  std::vector<int> hflags(count, 0);
  if (grouped) {
    IGAFD_BH(device_malloc((void**)&dflags, sizeof(int) * count));
    std::vector<int> all(count);
    for (int i = 0; i < count; ++i) all[i] = i;
    std::vector<GroupStep> ph;
    size_t foff = 0;
    for (int i = 0; i < count; ++i) {
      igafd_ctx* c = cs[i];
      SolverState init{};
      init.tol2 = o->rtol * o->rtol;
      init.maxit = maxit;
      init.flexible = o->flexible ? 1 : 0;
      *c->hstate = init;
      IGAFD_BH(hipMemcpyAsync(c->state, c->hstate, sizeof(SolverState), hipMemcpyHostToDevice, pool[0]));
    }
    IGAFD_BT(build_grouped_init(arena, ph, &foff, all, cs, bs, xs));
    IGAFD_BT(arena.upload(pool[0]));
    for (GroupStep& f : ph) IGAFD_BT(f(pool[0]));
    hipLaunchKernelGGL(k_gather_flags, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, pool[0],
                       arena.at<SolverState*>(foff), count, dflags);
    IGAFD_BH(hipGetLastError());
    IGAFD_BH(hipMemcpyAsync(hflags.data(), dflags, sizeof(int) * count, hipMemcpyDeviceToHost, pool[0]));
    IGAFD_BT(sync_all());
    std::vector<int> run;
    for (int i = 0; i < count; ++i) {
      z[i] = cs[i]->z;
      zold[i] = cs[i]->zold;
      running[i] = hflags[i] == FLAG_RUNNING;
      if (running[i]) run.push_back(i);
    }
    if (!run.empty()) {
      IGAFD_BT(build_grouped_start(arena, ph, run, cs, o->precision, Sp, z));
      IGAFD_BT(arena.upload(pool[0]));
      for (GroupStep& f : ph) IGAFD_BT(f(pool[0]));
    }
  } else {
    for (int i = 0; i < count; ++i) {
      igafd_ctx* c = cs[i];
      SolverState init{};
      init.tol2 = o->rtol * o->rtol;
      init.maxit = maxit;
      init.flexible = o->flexible ? 1 : 0;
      *c->hstate = init;
      IGAFD_BH(hipMemcpyAsync(c->state, c->hstate, sizeof(SolverState), hipMemcpyHostToDevice, c->stream));
      const unsigned vb = vblocks(c);
      hipLaunchKernelGGL(k_init, dim3(vb), dim3(kBlock), 0, c->stream, bs[i], nullptr, c->r, xs[i], 0, c->N,
                         c->partial);
      IGAFD_BH(hipGetLastError());
      IGAFD_BT(reduce(c, (int)vb, 1, RED_BB_RR, nullptr));
      IGAFD_BH(hipMemcpyAsync(c->hstate, c->state, sizeof(SolverState), hipMemcpyDeviceToHost, c->stream));
    }
    IGAFD_BT(sync_all());
    for (int i = 0; i < count; ++i) {
      igafd_ctx* c = cs[i];
      z[i] = c->z;
      zold[i] = c->zold;
      running[i] = c->hstate->flag == FLAG_RUNNING;
      if (running[i]) IGAFD_BT(start_directions(c, o->precision, Sp[i], z[i], zold[i]));
    }
  }
  const bool use_graph = std::getenv("IGAFD_NO_GRAPH") == nullptr;
  int captured_for = -1;
  double keep = 0.75;
  if (const char* e = std::getenv("IGAFD_BATCH_RECAPTURE")) keep = std::atof(e);
  if (grouped) {
    // the steps of `chunk` iterations (even: z / z_old return to their roles)
    // for the running set, captured once and replayed until the running count
    // falls below `keep` times the captured one
    std::vector<GroupStep> steps[2];
    std::vector<int> run, cap_run;
    size_t flags_off = 0;
    const hipStream_t gs = pool[0];
    auto enqueue = [&]() -> igafd_status {
      for (int k = 0; k < chunk; ++k)
        for (GroupStep& f : steps[k & 1]) IGAFD_TRY(f(gs));
      const int nc = (int)cap_run.size();
      hipLaunchKernelGGL(k_gather_flags, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, gs,
                         arena.at<SolverState*>(flags_off), nc, dflags);
      IGAFD_HIP_CHECK(hipGetLastError());
      return IGAFD_OK;
    };
    while (true) {
      run.clear();
      for (int i = 0; i < count; ++i)
        if (running[i]) run.push_back(i);
      if (run.empty()) break;
      const int nrun = (int)run.size();
      const bool rebuild = captured_for < 0 || nrun < keep * captured_for;
      if (rebuild) {
        if (exec) IGAFD_BH(hipGraphExecDestroy(exec));
        if (graph) IGAFD_BH(hipGraphDestroy(graph));
        exec = nullptr;
        graph = nullptr;
        IGAFD_BH(hipStreamSynchronize(gs));
        IGAFD_BT(build_grouped(arena, steps, &flags_off, run, cs, xs, o->precision, o->flexible ? 1 : 0, Sp, z, zold));
        IGAFD_BT(arena.upload(gs));
        cap_run = run;
        captured_for = nrun;
      }
      if (use_graph) {
        if (rebuild) {
          IGAFD_BH(hipStreamBeginCapture(gs, hipStreamCaptureModeRelaxed));
          st = enqueue();
          const hipError_t ec = hipStreamEndCapture(gs, &graph);
          if (st != IGAFD_OK) {
            cleanup();
            return st;
          }
          IGAFD_BH(ec);
          IGAFD_BH(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        }
        IGAFD_BH(hipGraphLaunch(exec, gs));
      } else {
        IGAFD_BT(enqueue());
      }
      IGAFD_BH(hipMemcpyAsync(hflags.data(), dflags, sizeof(int) * cap_run.size(), hipMemcpyDeviceToHost, gs));
      IGAFD_BH(hipStreamSynchronize(gs));
      for (size_t k = 0; k < cap_run.size(); ++k)
        running[cap_run[k]] = running[cap_run[k]] && hflags[k] == FLAG_RUNNING;
    }
  }
  // A graph captured for a set of running problems stays valid after some of
  // them converge (their kernels turn into no-ops on the device stop flag);
  // it is captured again only when the running count has fallen below
  // `keep` times the captured one, trading no-op launches against capture
  // and instantiation (a few ms for thousands of nodes).
  while (!grouped) {
    int nrun = 0;
    for (int i = 0; i < count; ++i) nrun += running[i];
    if (nrun == 0) break;
    auto enqueue_chunk = [&]() -> igafd_status {
      for (int k = 0; k < chunk; ++k)
        for (int i = 0; i < count; ++i)
          if (running[i])
            IGAFD_TRY(enqueue_iteration(cs[i], xs[i], o->precision, Sp[i], o->flexible ? 1 : 0, z[i], zold[i],
                                        nullptr));
      return IGAFD_OK;
    };
    if (use_graph) {
      if (captured_for < 0 || nrun < keep * captured_for) {  // (re)capture the chunk for the running set
        if (exec) IGAFD_BH(hipGraphExecDestroy(exec));
        if (graph) IGAFD_BH(hipGraphDestroy(graph));
        exec = nullptr;
        graph = nullptr;
        IGAFD_BT(sync_all());
        IGAFD_BH(hipStreamBeginCapture(pool[0], hipStreamCaptureModeRelaxed));
        IGAFD_BH(hipEventRecord(fork, pool[0]));
        for (int k = 1; k < nst; ++k) IGAFD_BH(hipStreamWaitEvent(pool[k], fork, 0));
        st = enqueue_chunk();
        for (int k = 1; k < nst; ++k) {
          (void)hipEventRecord(join[k], pool[k]);
          (void)hipStreamWaitEvent(pool[0], join[k], 0);
        }
        const hipError_t ec = hipStreamEndCapture(pool[0], &graph);
        if (st != IGAFD_OK) {
          cleanup();
          return st;
        }
        IGAFD_BH(ec);
        IGAFD_BH(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        captured_for = nrun;
      }
      IGAFD_BH(hipGraphLaunch(exec, pool[0]));
      for (int i = 0; i < count; ++i)
        IGAFD_BH(hipMemcpyAsync(cs[i]->hstate, cs[i]->state, sizeof(SolverState), hipMemcpyDeviceToHost, pool[0]));
    } else {
      IGAFD_BT(enqueue_chunk());
      for (int i = 0; i < count; ++i)
        IGAFD_BH(hipMemcpyAsync(cs[i]->hstate, cs[i]->state, sizeof(SolverState), hipMemcpyDeviceToHost,
                                cs[i]->stream));
    }
    IGAFD_BT(sync_all());
    for (int i = 0; i < count; ++i) running[i] = running[i] && cs[i]->hstate->flag == FLAG_RUNNING;
  }
  for (int k = 1; k < nst; ++k) IGAFD_BH(hipStreamWaitEvent(pool[0], join[k], 0));
  IGAFD_BH(hipEventRecord(t1, pool[0]));
  IGAFD_BT(sync_all());
  float ms = 0.f;
  IGAFD_BH(hipEventElapsedTime(&ms, t0, t1));
  if (wall_ms) *wall_ms = ms;
  // FP64 true residuals; a problem that misses the tolerance continues alone
  if (grouped) {
    std::vector<int> all(count);
    for (int i = 0; i < count; ++i) all[i] = i;
    std::vector<GroupStep> ph;
    IGAFD_BT(build_grouped_residual(arena, ph, all, cs, bs, xs));
    IGAFD_BT(arena.upload(pool[0]));
    for (GroupStep& f : ph) IGAFD_BT(f(pool[0]));
    for (int i = 0; i < count; ++i)
      IGAFD_BH(hipMemcpyAsync(cs[i]->hstate, cs[i]->state, sizeof(SolverState), hipMemcpyDeviceToHost, pool[0]));
  } else {
    for (int i = 0; i < count; ++i) {
      igafd_ctx* c = cs[i];
      const unsigned vb = vblocks(c);
      IGAFD_BT(spmv_unpadded(c, xs[i], c->q, nullptr, nullptr));
      hipLaunchKernelGGL(k_residual, dim3(vb), dim3(kBlock), 0, c->stream, bs[i], c->q, c->r, c->N, c->partial);
      IGAFD_BH(hipGetLastError());
      IGAFD_BT(reduce(c, (int)vb, 0, RED_TRUE, nullptr));
      IGAFD_BH(hipMemcpyAsync(c->hstate, c->state, sizeof(SolverState), hipMemcpyDeviceToHost, c->stream));
    }
  }
  IGAFD_BT(sync_all());
  for (int i = 0; i < count; ++i) {
    igafd_ctx* c = cs[i];
    const SolverState hs = *c->hstate;
    const double rel = hs.bb > 0.0 ? std::sqrt(hs.rrtrue / hs.bb) : 0.0;
    igafd_solve_info inf{};
    inf.iters = hs.iters;
    inf.relres = hs.bb > 0.0 ? std::sqrt(hs.rr / hs.bb) : 0.0;
    inf.true_relres = rel;
    inf.t_solve_ms = ms;
    inf.status = hs.flag == FLAG_BREAKDOWN ? IGAFD_ERR_BREAKDOWN : IGAFD_OK;
    if (!(rel <= o->rtol) && hs.flag != FLAG_BREAKDOWN) {
      igafd_solve_opts oc = *o;
      oc.use_x0 = 1;
      oc.maxit = maxit > hs.iters ? maxit - hs.iters : 1;
      oc.history = nullptr;
      oc.timers = 0;
      igafd_solve_info more{};
      const igafd_status s2 = solve_impl(c, bs[i], xs[i], &oc, &more);
      inf.iters = hs.iters + more.iters;
      inf.restarts = 1 + more.restarts;
      inf.true_relres = more.true_relres;
      inf.relres = more.relres;
      inf.status = s2;
    }
    if (infos) infos[i] = inf;
  }
  cleanup();
  for (int i = 0; i < count; ++i)
    if (infos && infos[i].status < 0) return (igafd_status)infos[i].status;
#undef IGAFD_BT
#undef IGAFD_BH
  return IGAFD_OK;
}

// Tile choice for one problem: time the FD apply for 1..4 row tiles per wave
// and the A product for 1, 2, 4 rows per thread; keep the fastest.
igafd_status autotune_impl(igafd_ctx* c, int reps) {
  IGAFD_HIP_CHECK(hipMemsetAsync(c->r, 0, sizeof(double) * c->N, c->stream));
  hipEvent_t a, b;
  IGAFD_HIP_CHECK(hipEventCreate(&a));
  IGAFD_HIP_CHECK(hipEventCreate(&b));
  auto time_it = [&](auto fn) -> float {
    fn();
    (void)hipEventRecord(a, c->stream);
    for (int k = 0; k < reps; ++k) fn();
    (void)hipEventRecord(b, c->stream);
    (void)hipEventSynchronize(b);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, a, b);
    return ms;
  };
  float best = 1e30f;
  int best_t = c->fd_tiles;
  for (int t = 1; t <= 4; ++t) {
    c->fd_tiles = t;
    const float ms = time_it([&]() { (void)fd_apply(c, IGAFD_FP64, c->r, c->z, nullptr, nullptr, nullptr); });
    if (ms < best) {
      best = ms;
      best_t = t;
    }
  }
  c->fd_tiles = best_t;
  // A product: the row-parallel kernel (1, 2, 4 rows per thread) and, in 3D,
  // the tiled kernel with the best tile shape for 64, 80 and 160 KB of LDS at
  // 256 threads per block and for 96, 128 and 160 KB at 512 (one block per CU:
  // larger tiles, fewer halo lines, but the grid's tail weighs more)
  struct Cand {
    int rows, b2, b3, tb;
  };
  std::vector<Cand> cands = {{1, 0, 0, 256}, {2, 0, 0, 256}, {4, 0, 0, 256}};
  int dev = 0, maxlds = 0;
  IGAFD_HIP_CHECK(hipGetDevice(&dev));
  IGAFD_HIP_CHECK(hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
  auto add = [&](long long lim, int tb) {
    int b2 = 0, b3 = 0;
    if (lim <= maxlds && spmv_pick_tile(c, lim, &b2, &b3, tb)) {
      bool seen = false;
      for (const Cand& k : cands) seen = seen || (k.b2 == b2 && k.b3 == b3 && k.tb == tb);
      if (!seen) cands.push_back({c->spmv_rows, b2, b3, tb});
    }
  };
  for (long long lim : {64LL * 1024, kTileLdsDefault, (long long)maxlds}) add(lim, 256);
  for (long long lim : {96LL * 1024, 128LL * 1024, (long long)maxlds}) add(lim, 512);
  best = 1e30f;
  Cand best_c{c->spmv_rows, c->tile_b2, c->tile_b3, c->tile_tb};
  for (const Cand& k : cands) {
    c->spmv_rows = k.rows;
    if (spmv_set_tile(c, k.b2, k.b3, k.tb) != IGAFD_OK) continue;
    bool ok = true;
    const float ms = time_it([&]() { ok = ok && spmv(c, c->pv, c->q, nullptr, nullptr) == IGAFD_OK; });
    // a later candidate must be 1% faster: near-ties keep the earlier one, so
    // repeated tunings of one problem settle on the same shape
    if (ok && ms < 0.99f * best) {
      best = ms;
      best_c = k;
    }
  }
  c->spmv_rows = best_c.rows;
  IGAFD_TRY(spmv_set_tile(c, best_c.b2, best_c.b3, best_c.tb));
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

}  // namespace
}  // namespace igafd

using namespace igafd;

namespace igafd {
namespace {
double elapsed_ms(std::chrono::steady_clock::time_point t0) {
  return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

// fd = false: no univariate eigendecompositions (a context whose
// preconditioner is applied by other contexts); with_A = false: no A and no
// CG workspace (a context that only applies P^-1)
igafd_status setup_impl(const igafd_problem* pr, void* stream, igafd_ctx** out, bool fd, bool with_A = true) {
  const auto t_start = std::chrono::steady_clock::now();
  if (!pr || !out) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  *out = nullptr;
  if (pr->dim != 2 && pr->dim != 3) {
    set_error("dim must be 2 or 3");
    return IGAFD_ERR_ARG;
  }
  std::unique_ptr<igafd_ctx, void (*)(igafd_ctx*)> c(new igafd_ctx(), igafd_destroy);
  c->dim = pr->dim;
  c->p = pr->degree;
  c->stream = (hipStream_t)stream;
  IGAFD_HIP_CHECK(hipGetDevice(&c->device));
  const int q = pr->quad_per_dir > 0 ? pr->quad_per_dir : pr->degree + 1;
  igafd_status s;
  if ((s = parse_geometry(pr, &c->geom)) != IGAFD_OK) return s;
  c->N = 1;
  for (int l = 0; l < pr->dim; ++l) {
    if ((s = build_direction(pr->degree, q, pr->nknots[l], pr->knots[l], &c->dir[l], false)) != IGAFD_OK) return s;
    c->n[l] = c->dir[l].n;
    c->N *= c->n[l];
  }
  for (int l = 0; l < pr->dim; ++l)
    if ((s = upload_tables(c->dir[l], &c->ddir[l], c->stream)) != IGAFD_OK) return s;
  // the univariate eigendecompositions and their copies (host)
  auto eigen = [&]() -> igafd_status {
    if (!fd) return IGAFD_OK;
    std::vector<Dir1D*> d;
    for (int l = 0; l < pr->dim; ++l) d.push_back(&c->dir[l]);
    igafd_status e = eigen_all(d);
    for (int l = 0; l < pr->dim && e == IGAFD_OK; ++l) e = upload_eigen(c->dir[l], &c->ddir[l], c->stream);
    return e;
  };
  if (with_A && c->dim == 3 && pr->want_features && (s = setup_modes(c.get())) != IGAFD_OK) return s;
  const int W = 2 * c->p + 1;
  const int Sz = (c->dim == 3) ? W * W * W : W * W;
  c->H = (Sz + 1) / 2;
  // zero halo: the largest stencil offset, rounded to 64 rows
  const long long maxoff = (long long)c->p * (1 + c->n[0] + (c->dim == 3 ? (long long)c->n[0] * c->n[1] : 0));
  c->halo = (maxoff + 63) / 64 * 64;
  c->Ns = (c->N + 2 * c->halo + 8 + 63) / 64 * 64;
  c->nnz = band_nnz(c.get());
  if (const char* e = std::getenv("IGAFD_SPMV_ROWS")) c->spmv_rows = std::atoi(e);
  if (const char* e = std::getenv("IGAFD_FD_TILES")) c->fd_tiles = std::atoi(e);
  if (c->fd_tiles < 1 || c->fd_tiles > 8) c->fd_tiles = 2;
  if (const char* e = std::getenv("IGAFD_FD_FUSED")) c->fd_fused = std::atoi(e) != 0;
  if (const char* e = std::getenv("IGAFD_FD_GEMM")) c->fd_gemm = std::atoi(e) != 0;
  if (!with_A) {
    // FD intermediates (FP64 is the widest) and the block partials of the
    // preconditioner's (r, s) product and of the spectral bounds
    if ((s = alloc_scratch(c.get(), {&c->fdbuf[0], &c->fdbuf[1]})) != IGAFD_OK) return s;
    c->npartial = partial_capacity(c.get());
    IGAFD_HIP_CHECK(device_malloc((void**)&c->partial, sizeof(double) * 2 * (size_t)c->npartial));
    if ((s = eigen()) != IGAFD_OK) return s;
    IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
    c->t_setup_ms = elapsed_ms(t_start);
    *out = c.release();
    return IGAFD_OK;
  }
  if ((s = block_alloc((void**)&c->band, sizeof(double) * (size_t)c->H * (size_t)c->Ns)) != IGAFD_OK) return s;
  if ((s = alloc_workspace(c.get())) != IGAFD_OK) return s;
  {
    // 3D: tiled A product by default (IGAFD_SPMV_TILE=0 selects the row-parallel
    // kernel, IGAFD_SPMV_TILE=<b2>x<b3>[x<threads per block>] a tile shape)
    int b2 = 0, b3 = 0, tb = 256;
    const char* e = std::getenv("IGAFD_SPMV_TILE");
    if (e && std::strchr(e, 'x')) {
      const char* e3 = std::strchr(e, 'x') + 1;
      b2 = std::atoi(e);
      b3 = std::atoi(e3);
      if (std::strchr(e3, 'x')) tb = std::atoi(std::strchr(e3, 'x') + 1);
    } else if (!(e && std::atoi(e) == 0)) {
      int dev = 0, maxlds = 0;
      IGAFD_HIP_CHECK(hipGetDevice(&dev));
      IGAFD_HIP_CHECK(hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
      double s256 = 0.0, s512 = 0.0;
      int c2 = 0, c3 = 0;
      if (!spmv_pick_tile(c.get(), kTileLdsDefault, &b2, &b3, 256, &s256)) b2 = b3 = 0;
      if (c->p >= 1 && c->p <= 6 && kTile512Default[c->p] &&
          spmv_pick_tile(c.get(), std::min(kTile512Lds, (long long)maxlds), &c2, &c3, 512, &s512) && s512 > s256) {
        b2 = c2;
        b3 = c3;
        tb = 512;
      }
    }
    if ((s = spmv_set_tile(c.get(), b2, b3, tb)) != IGAFD_OK) return s;
  }
  // the device assembles A while the host computes the eigendecompositions
  AsmWork work{nullptr, c.get()};
  s = assemble_band(c.get(), pr->want_features != 0, &work);
  const igafd_status se = s == IGAFD_OK ? eigen() : s;
  if (se != IGAFD_OK) return se;
  if ((s = assemble_finish(c.get())) != IGAFD_OK) return s;
  c->t_setup_ms = elapsed_ms(t_start);
  *out = c.release();
  return IGAFD_OK;
}

igafd_status lshape_setup_impl(int degree, int nknots, const double* knots, void* stream, igafd_ctx** out) {
  const auto t_start = std::chrono::steady_clock::now();
  if (!knots || !out) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  *out = nullptr;
  const int p = degree;
  Dir1D patch;
  igafd_status s;
  if ((s = build_direction(p, p + 1, nknots, knots, &patch, false)) != IGAFD_OK) return s;
  // the knot vector of two patches side by side: the patch knots on [0,1/2]
  // and on [1/2,1], joined by a knot of multiplicity p at 1/2 (C^0)
  std::vector<double> km;
  km.assign(p + 1, 0.0);
  for (int i = p + 1; i < nknots - p - 1; ++i) km.push_back(0.5 * knots[i]);
  km.insert(km.end(), p, 0.5);
  for (int i = p + 1; i < nknots - p - 1; ++i) km.push_back(0.5 + 0.5 * knots[i]);
  km.insert(km.end(), p + 1, 1.0);
  igafd_problem pr{};
  pr.dim = 2;
  pr.degree = p;
  pr.nknots[0] = pr.nknots[1] = (int)km.size();
  pr.knots[0] = pr.knots[1] = km.data();
  pr.geom_kind = IGAFD_GEOM_IDENTITY;
  pr.coef_kind = IGAFD_COEF_ONE;
  pr.quad_per_dir = p + 1;
  igafd_ctx* raw = nullptr;
  if ((s = setup_impl(&pr, stream, &raw, false)) != IGAFD_OK) return s;
  std::unique_ptr<igafd_ctx, void (*)(igafd_ctx*)> c(raw, igafd_destroy);
  const int h = patch.n;
  if (c->n[0] != 2 * h + 1 || c->n[1] != 2 * h + 1) {
    set_error("internal: bounding-square grid does not match the patches");
    return IGAFD_ERR_ARG;
  }
  // Theta_1 = the corner patch and the one above it: one patch along
  // direction 1, two along direction 2; Theta_2 = the corner patch and the one
  // to its right
  Dir1D merged;
  if ((s = build_direction(p, p + 1, (int)km.size(), km.data(), &merged, false)) != IGAFD_OK) return s;
  if ((s = eigen_all({&patch, &merged})) != IGAFD_OK) return s;
  if ((s = create_fd_sub(p, patch, merged, c->stream, &c->sub[0])) != IGAFD_OK) return s;
  if ((s = create_fd_sub(p, merged, patch, c->stream, &c->sub[1])) != IGAFD_OK) return s;
  c->hole = h;
  IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
  c->t_setup_ms = elapsed_ms(t_start);
  *out = c.release();
  return IGAFD_OK;
}
}  // namespace
}  // namespace igafd

extern "C" {

const char* igafd_last_error(void) { return g_err.c_str(); }

igafd_status igafd_univariate(int degree, int nknots, const double* knots, int quad, double* M, double* K, double* U,
                              double* lam, int* n_out) {
  return guarded([&]() -> igafd_status {
    Dir1D d;
    const int q = quad > 0 ? quad : degree + 1;
    igafd_status s = build_direction(degree, q, nknots, knots, &d);
    if (s != IGAFD_OK) return s;
    if (n_out) *n_out = d.n;
    if (M) std::memcpy(M, d.M.data(), sizeof(double) * d.M.size());
    if (K) std::memcpy(K, d.K.data(), sizeof(double) * d.K.size());
    if (U) std::memcpy(U, d.U.data(), sizeof(double) * d.U.size());
    if (lam) std::memcpy(lam, d.lam.data(), sizeof(double) * d.lam.size());
    return IGAFD_OK;
  });
}

long long igafd_release_cached(void) {
  std::lock_guard<std::mutex> lock(g_block_mutex);
  long long bytes = 0;
  for (const Block& b : g_cached) {
    (void)hipFree(b.p);
    bytes += (long long)b.bytes;
  }
  g_cached.clear();
  return bytes;
}

void igafd_destroy(igafd_ctx* c) {
  if (!c) return;
  const bool idle = wait_stream(c->stream, c->device);  // its blocks may go to another context and stream
  for (int k = 0; k < 2; ++k) igafd_destroy(c->sub[k]);
  adi_free(c);
  for (int l = 0; l < 3; ++l) free_dir(&c->ddir[l]);
  for (double* b : {c->band, c->ext, c->scratch, c->pv_pad, c->xpad, c->scaling}) block_free(b, idle);
  block_free(c->feat, idle);
  free_dev(c->partial);
  free_dev(c->state);
  free_dev(c->dflag);
  if (c->hstate) (void)hipHostFree(c->hstate);
  if (c->ev0) (void)hipEventDestroy(c->ev0);
  if (c->ev1) (void)hipEventDestroy(c->ev1);
  free_dev(c->hist);
  free_dev(c->modes);
  for (hipEvent_t e : c->tev) (void)hipEventDestroy(e);
  delete c;
}


igafd_status igafd_setup(const igafd_problem* pr, void* stream, igafd_ctx** out) {
  return guarded([&]() { return setup_impl(pr, stream, out, true); });
}

igafd_status igafd_setup_precond(const igafd_problem* pr, void* stream, igafd_ctx** out) {
  return guarded([&]() { return setup_impl(pr, stream, out, true, false); });
}

igafd_status igafd_lshape_setup(int degree, int nknots, const double* knots, void* stream, igafd_ctx** out) {
  return guarded([&]() { return lshape_setup_impl(degree, nknots, knots, stream, out); });
}

}  // extern "C"

namespace igafd {
namespace {
igafd_status set_adi_impl(igafd_ctx* c, double eps, int rule, int* J, double* rho) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (eps == 0.0) {
    adi_free(c);
    if (J) *J = 0;
    if (rho) *rho = 0.0;
    return IGAFD_OK;
  }
  if (c->hole >= 0) {
    set_error("the ADI preconditioner is for single-patch 3D problems");
    return IGAFD_ERR_ARG;
  }
  const igafd_status s = adi_setup(c, eps, rule);
  if (s != IGAFD_OK) return s;
  if (J) *J = (int)c->adi->omega.size();
  if (rho) *rho = c->adi->rho;
  return IGAFD_OK;
}
}  // namespace
}  // namespace igafd

extern "C" {

igafd_status igafd_set_adi(igafd_ctx* c, double eps, int* J, double* rho) {
  return guarded([&]() { return set_adi_impl(c, eps, kAdiGeometric, J, rho); });
}

igafd_status igafd_set_adi_greedy(igafd_ctx* c, double eps, int* J, double* rho) {
  return guarded([&]() { return set_adi_impl(c, eps, kAdiGreedy, J, rho); });
}

igafd_status igafd_get_adi(const igafd_ctx* c, int* J, int* J0, double* rho, double* omegas, int capacity) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (!c->adi) {
    if (J) *J = 0;
    if (J0) *J0 = 0;
    if (rho) *rho = 0.0;
    return IGAFD_OK;
  }
  const int n = (int)c->adi->omega.size();
  if (omegas && capacity < n) {
    set_error("omega array too short");
    return IGAFD_ERR_ARG;
  }
  if (J) *J = n;
  if (J0) *J0 = c->adi->J0;
  if (rho) *rho = c->adi->rho;
  if (omegas) std::memcpy(omegas, c->adi->omega.data(), sizeof(double) * n);
  return IGAFD_OK;
}

igafd_status igafd_lshape_corner(const igafd_ctx* c, int* hole, long long* ndofs) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  const long long w = c->hole >= 0 ? c->n[0] - c->hole : 0;
  if (hole) *hole = c->hole;
  if (ndofs) *ndofs = c->N - w * w;
  return IGAFD_OK;
}

igafd_status igafd_sizes(const igafd_ctx* c, int n[3], long long* N, long long* nnz, long long* band_bytes) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (n)
    for (int l = 0; l < 3; ++l) n[l] = c->n[l];
  if (N) *N = c->N;
  if (nnz) *nnz = c->nnz;
  if (band_bytes) *band_bytes = c->band ? (long long)sizeof(double) * c->H * c->Ns : 0;
  return IGAFD_OK;
}

igafd_status igafd_load_vector(igafd_ctx* c, int rhs_kind, const double* rhs_params, int n_rhs_params, double* b) {
  if (!c || !b) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  const igafd_status s = assemble_load(c, rhs_kind, rhs_params, n_rhs_params, b);
  return s == IGAFD_OK ? mask_hole(c, b) : s;
}

igafd_status igafd_apply_A(igafd_ctx* c, const double* x, double* y) {
  if (!c || !x || !y || x == y) {
    set_error("apply_A needs distinct non-null vectors");
    return IGAFD_ERR_ARG;
  }
  if (no_A(c, "igafd_apply_A")) return IGAFD_ERR_ARG;
  return spmv_unpadded(c, x, y, nullptr, nullptr);
}

igafd_status igafd_apply_precond(igafd_ctx* c, int precision, const double* r, double* s) {
  if (!c || !r || !s || r == s) {
    set_error("apply_precond needs distinct non-null vectors");
    return IGAFD_ERR_ARG;
  }
  return fd_apply(c, precision, r, s, c->scaling_set ? c->scaling : nullptr, nullptr, nullptr);
}

igafd_status igafd_set_scaling(igafd_ctx* c, const double* S) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (!S) {
    c->scaling_set = false;
    return IGAFD_OK;
  }
  if (is_lshape(c, "the scaled preconditioner")) return IGAFD_ERR_ARG;
  if (!c->scaling && block_alloc((void**)&c->scaling, sizeof(double) * c->N) != IGAFD_OK) return IGAFD_ERR_HIP;
  IGAFD_HIP_CHECK(hipMemcpyAsync(c->scaling, S, sizeof(double) * c->N, hipMemcpyDeviceToDevice, c->stream));
  c->scaling_set = true;
  return IGAFD_OK;
}

igafd_status igafd_diagonals(igafd_ctx* c, double* dA, double* dP) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_diagonals")) return IGAFD_ERR_ARG;
  if (no_A(c, "igafd_diagonals")) return IGAFD_ERR_ARG;
  return diagonals(c, dA, dP);
}

igafd_status igafd_features(igafd_ctx* c, float* feat) {
  if (!c || !feat) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_features")) return IGAFD_ERR_ARG;
  if (no_A(c, "igafd_features")) return IGAFD_ERR_ARG;
  return features(c, feat);
}

}  // extern "C"

namespace igafd {
namespace {
// Accumulator of igafd_features_noalloc: 8 doubles per dof for N <= 2^20
// (64 MiB), a file-scope device array that every GPU the library runs on
// holds from module load until the process ends.  Host code never passes
// `scratch` itself (on the host that name is only a stand-in): the device
// address comes from hipGetSymbolAddress, looked up once per device.
constexpr long long kScratchDofs = 1LL << 20;
__device__ __align__(256) double scratch[8 * kScratchDofs];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// device address of `scratch` on device `dev` (the current device)
igafd_status scratch_address(int dev, double** out) {
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("device ordinal out of range for the static accumulator");
    return IGAFD_ERR_ARG;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    double* p = nullptr;
    IGAFD_HIP_CHECK(hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch)));
    if (!p) {
      set_error("hipGetSymbolAddress returned no address for the static accumulator");
      return IGAFD_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return IGAFD_OK;
}
}  // namespace
}  // namespace igafd

extern "C" {

igafd_status igafd_features_noalloc(igafd_ctx* c, float* feat) {
  if (!c || !feat) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_features_noalloc")) return IGAFD_ERR_ARG;
  if (no_A(c, "igafd_features_noalloc")) return IGAFD_ERR_ARG;
  if (c->feat) {  // assembled with A at setup: a device copy
    IGAFD_HIP_CHECK(
        hipMemcpyAsync(feat, c->feat, sizeof(float) * 8 * (size_t)c->N, hipMemcpyDeviceToDevice, c->stream));
    return IGAFD_OK;
  }
  if (c->N > kScratchDofs) {
    set_error("igafd_features_noalloc: N = " + std::to_string(c->N) + " exceeds the static accumulator (" +
              std::to_string(kScratchDofs) + " dofs); use igafd_features or set up with want_features");
    return IGAFD_ERR_ARG;
  }
  int dev = -1;
  IGAFD_HIP_CHECK(hipGetDevice(&dev));
  if (dev != c->device) {
    set_error("igafd_features_noalloc: the context's device must be current");
    return IGAFD_ERR_ARG;
  }
  double* acc = nullptr;
  IGAFD_TRY(scratch_address(dev, &acc));
  return features_into(c, acc, feat);
}

igafd_status igafd_scaling_targets(igafd_ctx* c, float* t) {
  if (!c || !t) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_scaling_targets")) return IGAFD_ERR_ARG;
  if (no_A(c, "igafd_scaling_targets")) return IGAFD_ERR_ARG;
  return scaling_targets(c, t);
}

igafd_status igafd_set_scaling_diag_ratio(igafd_ctx* c) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "the scaled preconditioner")) return IGAFD_ERR_ARG;
  if (no_A(c, "igafd_set_scaling_diag_ratio")) return IGAFD_ERR_ARG;
  if (!c->scaling && block_alloc((void**)&c->scaling, sizeof(double) * c->N) != IGAFD_OK) return IGAFD_ERR_HIP;
  igafd_status st = diag_ratio_scaling(c, c->scaling);
  if (st == IGAFD_OK) c->scaling_set = true;
  return st;
}

igafd_status igafd_get_eigen(const igafd_ctx* c, int dir, double* U, double* lam) {
  if (!c || dir < 0 || dir >= c->dim) {
    set_error("bad context or direction");
    return IGAFD_ERR_ARG;
  }
  const Dir1D& d = c->dir[dir];
  if (d.U.empty()) {
    set_error("this context holds no univariate eigendecomposition (L-shaped multi-patch context)");
    return IGAFD_ERR_ARG;
  }
  if (U) std::memcpy(U, d.U.data(), sizeof(double) * d.U.size());
  if (lam) std::memcpy(lam, d.lam.data(), sizeof(double) * d.lam.size());
  return IGAFD_OK;
}

igafd_status igafd_solve_batched(igafd_ctx* const* ctxs, int count, const double* const* b, double* const* u,
                                 const igafd_solve_opts* o, igafd_solve_info* infos, double* wall_ms) {
  if (!ctxs || !b || !u || !o || count < 1) {
    set_error("batched solve needs count >= 1 contexts, vectors and options");
    return IGAFD_ERR_ARG;
  }
  for (int i = 0; i < count; ++i) {
    if (ctxs[i] && is_lshape(ctxs[i], "igafd_solve_batched")) return IGAFD_ERR_ARG;
    if (ctxs[i] && no_A(ctxs[i], "igafd_solve_batched")) return IGAFD_ERR_ARG;
    if (ctxs[i] && ctxs[i]->adi) {
      set_error("igafd_solve_batched runs the FD preconditioner only");
      return IGAFD_ERR_ARG;
    }
  }
  return solve_batched_impl(ctxs, count, b, u, o, infos, wall_ms);
}

igafd_status igafd_spectral_bounds(igafd_ctx* c, double* qmin, double* qmax, double* qloc) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_spectral_bounds")) return IGAFD_ERR_ARG;
  return spectral_bounds(c, qmin, qmax, qloc);
}

igafd_status igafd_scaling_gate(igafd_ctx* c, double gain, int* use, double* kappa_q, double* kappa_loc) {
  if (!c || !(gain > 0.0)) {
    set_error("scaling gate needs a context and a positive gain");
    return IGAFD_ERR_ARG;
  }
  if (is_lshape(c, "igafd_scaling_gate")) return IGAFD_ERR_ARG;
  return gate_impl(c, gain, use, kappa_q, kappa_loc);
}

igafd_status igafd_get_shape(const igafd_ctx* c, int* spmv_rows, int* tile_b2, int* tile_b3, int* fd_fused,
                             int* fd_tiles, int* tile_threads) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (spmv_rows) *spmv_rows = c->spmv_rows;
  if (tile_b2) *tile_b2 = c->tile_b2;
  if (tile_b3) *tile_b3 = c->tile_b3;
  if (fd_fused) *fd_fused = (c->fd_fused && fd_fused_ok(c)) ? 1 : 0;
  if (fd_tiles) *fd_tiles = c->fd_tiles;
  if (tile_threads) *tile_threads = c->tile_tb;
  return IGAFD_OK;
}

igafd_status igafd_autotune(igafd_ctx* c, int fd_tiles, int spmv_rows) {
  if (!c) {
    set_error("null context");
    return IGAFD_ERR_ARG;
  }
  if (fd_tiles > 0 || spmv_rows > 0) {  // explicit choice
    if (fd_tiles > 8 || spmv_rows > 4 || spmv_rows == 3) {
      set_error("fd_tiles must be 1..8 and spmv_rows 1, 2 or 4");
      return IGAFD_ERR_ARG;
    }
    if (fd_tiles > 0) c->fd_tiles = fd_tiles;
    if (spmv_rows > 0) {
      if (no_A(c, "the A-product shape")) return IGAFD_ERR_ARG;
      c->spmv_rows = spmv_rows;
      return spmv_set_tile(c, 0, 0);  // an explicit row count selects the row-parallel kernel
    }
    return IGAFD_OK;
  }
  if (no_A(c, "igafd_autotune")) return IGAFD_ERR_ARG;
  return autotune_impl(c, 8);
}

igafd_status igafd_solve(igafd_ctx* c, const double* b, double* u, const igafd_solve_opts* o, igafd_solve_info* info) {
  if (!c || !b || !u || !o || b == u) {
    set_error("solve needs a context, distinct b and u, and options");
    return IGAFD_ERR_ARG;
  }
  if (no_A(c, "igafd_solve")) return IGAFD_ERR_ARG;
  return solve_impl(c, b, u, o, info);
}

}  // extern "C"
