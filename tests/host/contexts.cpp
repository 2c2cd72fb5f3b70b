// Contexts on the host runtime of hip_double.h.  The argument names a check;
// prints "OK" and returns 0 when it holds.
#include <sys/syscall.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "hip_double.h"
#include "internal.h"

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::printf("FAILED line %d: %s\n", __LINE__, #x);     \
      return 1;                                              \
    }                                                        \
  } while (0)

namespace {
std::atomic<int> yielded{0};
}

// Host allocations: while `fail_at` is not negative, the allocation of that
// number (counted over all threads) fails.
namespace {
std::atomic<long long> fail_at{-1}, allocations{0};

void* host_alloc(size_t n) {
  if (fail_at >= 0 && !hip_double::inside && allocations++ == fail_at) return nullptr;
  return std::malloc(n ? n : 1);
}
}  // namespace
void* operator new(size_t n) {
  if (void* p = host_alloc(n)) return p;
  throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return host_alloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// counts the threads that have waited at a barrier long enough to yield
extern "C" int sched_yield(void) noexcept {
  static thread_local bool counted = false;
  if (!counted) yielded += 1;
  counted = true;
  return (int)syscall(SYS_sched_yield);
}

namespace {

std::vector<double> knots(int E, int p) {
  std::vector<double> k(p + 1, 0.0);
  for (int e = 1; e < E; ++e) k.push_back((double)e / E);
  k.insert(k.end(), p + 1, 1.0);
  return k;
}

igafd_ctx* setup(int E, int p, hipStream_t st, bool features = false) {
  const std::vector<double> k = knots(E, p);
  igafd_problem pr{};
  pr.dim = 3;
  pr.degree = p;
  for (int l = 0; l < 3; ++l) {
    pr.nknots[l] = (int)k.size();
    pr.knots[l] = k.data();
  }
  pr.geom_kind = IGAFD_GEOM_RING;
  pr.want_features = features;
  igafd_ctx* c = nullptr;
  if (igafd_setup(&pr, st, &c) != IGAFD_OK) std::printf("%s\n", igafd_last_error());
  return c;
}

bool waited(int device, hipStream_t st) {
  for (const hip_double::Sync& s : hip_double::syncs)
    if (s.device == device && (s.stream == st || s.stream == hip_double::kWhole)) return true;
  return false;
}

// The memory of a destroyed context goes to later contexts: its device and
// stream have to be waited for, whichever device is current.
int destroy_waits() {
  CHECK(hipSetDevice(1) == hipSuccess);
  igafd_ctx* c = setup(24, 3, nullptr);
  CHECK(c);
  CHECK(hipSetDevice(0) == hipSuccess);
  hip_double::forget();
  igafd_destroy(c);
  CHECK(waited(1, nullptr));
  int d = -1;
  CHECK(hipGetDevice(&d) == hipSuccess && d == 0);
  // the L-shaped context's subdomains live on the same device
  CHECK(hipSetDevice(1) == hipSuccess);
  const std::vector<double> k = knots(200, 2);
  CHECK(igafd_lshape_setup(2, (int)k.size(), k.data(), nullptr, &c) == IGAFD_OK);
  CHECK(hipSetDevice(0) == hipSuccess);
  hip_double::forget();
  igafd_destroy(c);
  for (const hip_double::Sync& s : hip_double::syncs) CHECK(s.device == 1);
  CHECK(waited(1, nullptr));
  return 0;
}

// A stream that was destroyed before its context cannot be waited for: the
// device is; where that fails too, nothing may be handed to another context.
int destroyed_stream() {
  hipStream_t st = (hipStream_t)0x1000;
  igafd_ctx* c = setup(24, 3, st);
  CHECK(c);
  hip_double::dead = st;
  hip_double::forget();
  igafd_destroy(c);
  CHECK(waited(0, hip_double::kWhole));
  hip_double::dead = nullptr;
  c = setup(24, 3, st);
  CHECK(c);
  hip_double::dead = st;
  hip_double::device_lost = true;
  igafd_destroy(c);
  CHECK(hip_double::bytes_on(0) == 0);
  return 0;
}

// Three different directions of 600 unknowns and more: the threads that wait at
// the barriers of their decompositions, which run at once, stay within one budget.
int eigen_budget() {
  std::vector<double> k[3];
  igafd_problem pr{};
  pr.dim = 3;
  pr.degree = 2;
  for (int l = 0; l < 3; ++l) {
    k[l] = knots(600 + l, 2);
    pr.nknots[l] = (int)k[l].size();
    pr.knots[l] = k[l].data();
  }
  igafd_ctx* c = nullptr;
  CHECK(igafd_setup_precond(&pr, nullptr, &c) == IGAFD_OK);
  igafd_destroy(c);
  const int budget = std::max(3, std::min(16, (int)std::thread::hardware_concurrency()));
  std::printf("%d threads at barriers, budget %d\n", yielded.load(), budget);
  CHECK(yielded <= budget);
  return 0;
}

// Each host allocation of a call in turn fails: the call reports it, leaves no
// device memory behind, and the next call works.
template <class F>
int each_allocation_fails(const F& call, long long stride) {
  for (long long k = 0;; k += stride) {
    igafd_ctx* c = nullptr;
    allocations = 0;
    fail_at = k;
    const igafd_status st = call(&c);
    const bool hit = allocations > k;
    fail_at = -1;
    CHECK(st == IGAFD_OK || st == IGAFD_ERR_ALLOC);
    CHECK(hit || st == IGAFD_OK);
    CHECK((st == IGAFD_OK) == (c != nullptr));
    if (st == IGAFD_ERR_ALLOC) CHECK(std::string(igafd_last_error()) == "out of host memory");
    igafd_destroy(c);
    igafd_release_cached();
    CHECK(hip_double::live.empty());
    if (!hit) {
      std::printf("%lld allocations\n", allocations.load());
      return 0;
    }
  }
}

int host_memory() {
  std::vector<double> k[3];
  igafd_problem pr{};
  pr.degree = 2;
  auto sizes = [&](std::vector<int> E) {
    pr.dim = (int)E.size();
    for (int l = 0; l < pr.dim; ++l) {
      k[l] = knots(E[l], 2);
      pr.nknots[l] = (int)k[l].size();
      pr.knots[l] = k[l].data();
    }
  };
  sizes({24, 25, 26});
  pr.want_features = 1;
  if (each_allocation_fails([&](igafd_ctx** c) { return igafd_setup(&pr, nullptr, c); }, 1)) return 1;
  sizes({40, 300, 20});  // its rotations are applied by several threads
  if (each_allocation_fails([&](igafd_ctx** c) { return igafd_setup_precond(&pr, nullptr, c); }, 5)) return 1;
  sizes({601, 600});     // thread teams
  if (each_allocation_fails([&](igafd_ctx** c) { return igafd_setup_precond(&pr, nullptr, c); }, 7)) return 1;
  sizes({20, 21});
  if (each_allocation_fails(
          [&](igafd_ctx** c) { return igafd_lshape_setup(2, pr.nknots[0], pr.knots[0], nullptr, c); }, 1))
    return 1;
  return 0;
}

// The dynamic LDS a function may use is the same for every problem: set to what
// one problem needs, it could be lowered by one thread's setup between the
// setting and the launch of another's.
int lds_limits() {
  const std::vector<double> k = knots(12, 3);
  hip_double::forget();
  for (int modes : {16, 4, 1}) {
    std::vector<double> g = {0.01, (double)modes};
    for (int i = 0; i < 3 * modes; ++i) g.push_back(0.1);
    for (int i = 0; i < 3 * modes; ++i) g.push_back(1.0 + i % 2);
    igafd_problem pr{};
    pr.dim = 3;
    pr.degree = 3;
    for (int l = 0; l < 3; ++l) {
      pr.nknots[l] = (int)k.size();
      pr.knots[l] = k.data();
    }
    pr.geom_kind = IGAFD_GEOM_WARPED;
    pr.geom_params = g.data();
    pr.n_geom_params = (int)g.size();
    pr.want_features = 1;
    igafd_ctx* c = nullptr;
    CHECK(igafd_setup(&pr, nullptr, &c) == IGAFD_OK);
    igafd_destroy(c);
  }
  for (int E : {128, 120, 112, 104, 96, 88}) {  // tiled A products of one degree, different tiles
    igafd_ctx* c = setup(E, 3, nullptr);
    CHECK(c && igafd_apply_A(c, c->r, c->z) == IGAFD_OK);
    igafd_destroy(c);
  }
  CHECK(!hip_double::attrs.empty());
  for (const hip_double::Attr& a : hip_double::attrs)
    for (const hip_double::Attr& b : hip_double::attrs) CHECK(a.fn != b.fn || a.value == b.value);
  CHECK(!hip_double::over_limit);
  return 0;
}

// The ADI sub-steps take half the lines per block where 32 would not all be
// resident at once: by the device's compute units.
int adi_lines() {
  hip_double::cus = 32;  // a partition of the card
  igafd_ctx c;
  c.dim = 3;
  c.p = 3;
  c.n[0] = c.n[1] = c.n[2] = 97;
  c.N = 97LL * 97 * 97;
  c.npartial = igafd::partial_capacity(&c);
  CHECK(igafd::adi_dot_blocks(&c) == (97 * 97 + 15) / 16);
  c.n[0] = c.n[1] = 20;  // 400 lines: 13 blocks of 32
  c.N = 400LL * 97;
  CHECK(igafd::adi_dot_blocks(&c) == 13);
  return 0;
}

// Switching to ADI takes one allocation for its tables and one for its vectors,
// and raises the LDS limits of the sub-steps that need it only.
int adi_setup() {
  igafd_ctx* c = setup(20, 3, nullptr);
  CHECK(c);
  const size_t before = hip_double::live.size();
  hip_double::forget();
  int J = 0;
  double rho = 0.0;
  CHECK(igafd_set_adi(c, 0.1, &J, &rho) == IGAFD_OK && J > 1);
  CHECK(hip_double::live.size() == before + 2);
  CHECK(hip_double::attrs.empty());
  CHECK(igafd_set_adi_greedy(c, 0.1, &J, &rho) == IGAFD_OK);  // the tables of the other rule go
  CHECK(hip_double::live.size() == before + 2);
  CHECK(igafd_set_adi(c, 0.0, &J, &rho) == IGAFD_OK && hip_double::live.size() == before);
  igafd_destroy(c);
  c = setup(95, 3, nullptr);
  hip_double::forget();
  CHECK(c && igafd_set_adi(c, 0.1, &J, &rho) == IGAFD_OK && !hip_double::attrs.empty());
  CHECK(igafd_apply_precond(c, IGAFD_FP64, c->r, c->z) == IGAFD_OK && !hip_double::over_limit);
  igafd_destroy(c);
  return 0;
}

// A tile shape whose accumulators find no room leaves the context with the
// row-parallel A product, not with the old shape and no accumulators.
int tile_without_room() {
  igafd_ctx* c = setup(64, 3, nullptr);
  CHECK(c && c->tile_b2 > 0 && c->ext);
  const int b2 = c->tile_b2, b3 = c->tile_b3, tb = c->tile_tb;
  const size_t held = hip_double::bytes_on(0);
  igafd::block_free(c->ext, false);  // as a larger shape does before it asks
  c->ext = nullptr;
  c->ext_cap = 0;
  hip_double::capacity = hip_double::bytes_on(0) + 1000;
  CHECK(igafd::spmv_set_tile(c, b2, b3, tb) != IGAFD_OK);
  CHECK(c->tile_b2 == 0 && !c->ext);
  CHECK(igafd_apply_A(c, c->r, c->z) == IGAFD_OK);
  hip_double::capacity = held + (64 << 20);
  CHECK(igafd::spmv_set_tile(c, b2, b3, tb) == IGAFD_OK && c->ext && c->tile_b2 == b2);
  igafd_destroy(c);
  return 0;
}

// Each device allocation of a sequence of calls fails in turn (and the second
// try with it): a status, no use of what is not there, and nothing left behind.
int device_memory() {
  const std::vector<double> k = knots(30, 3);
  for (long long f = 0;; ++f) {
    hip_double::device_allocs = 0;
    hip_double::fail_alloc = f;
    igafd_ctx* c = setup(30, 3, nullptr, true);
    igafd_ctx* d = nullptr;
    (void)igafd_lshape_setup(3, (int)k.size(), k.data(), nullptr, &d);
    if (c) {
      double* x = c->r;
      (void)igafd_set_scaling(c, x);
      (void)igafd_set_scaling_diag_ratio(c);
      int J = 0;
      (void)igafd_set_adi_greedy(c, 0.1, &J, nullptr);
      (void)igafd_apply_precond(c, IGAFD_FP64, c->r, c->z);
      (void)igafd_set_adi(c, 0.0, nullptr, nullptr);
      (void)igafd_autotune(c, 0, 0);
      CHECK(c->tile_b2 == 0 || c->ext);
      (void)igafd_apply_A(c, c->q, c->z);
      (void)igafd_load_vector(c, IGAFD_RHS_ONE, nullptr, 0, c->q);
    }
    igafd_destroy(c);
    igafd_destroy(d);
    const bool hit = hip_double::device_allocs > f;
    hip_double::fail_alloc = -1;
    igafd_release_cached();
    CHECK(hip_double::live.empty());
    (void)hipGetLastError();
    if (!hit) {
      std::printf("%lld device allocations\n", hip_double::device_allocs);
      return 0;
    }
  }
}

constexpr size_t kMiB = 1 << 20, kGiB = (size_t)1 << 30;

void* take(size_t bytes) {
  void* p = nullptr;
  return igafd::block_alloc(&p, bytes) == IGAFD_OK ? p : nullptr;
}

// Reuse: by device, for requests of 4/5 of a block and more, the smallest such
// block first; small blocks are not kept.
int cache_fit() {
  void* a = take(100 * kMiB);
  void* b = take(90 * kMiB);
  CHECK(a && b);
  igafd::block_free(a);
  igafd::block_free(b);
  CHECK(hip_double::frees == 0);
  CHECK(take(80 * kMiB) == b);
  CHECK(take(80 * kMiB) == a);
  igafd::block_free(a);
  void* c = take(79 * kMiB);  // below 4/5
  CHECK(c && c != a);
  CHECK(take(101 * kMiB) != a);
  CHECK(hipSetDevice(1) == hipSuccess);
  void* d = take(100 * kMiB);
  CHECK(d != a && hip_double::bytes_on(1) == 100 * kMiB);
  igafd::block_free(d);  // freed from any device, reused on its own
  CHECK(hipSetDevice(0) == hipSuccess);
  CHECK(take(100 * kMiB) == a);
  CHECK(take(100 * kMiB) != d);
  void* s = take(kMiB - 1);
  const long long frees = hip_double::frees;
  igafd::block_free(s);
  CHECK(hip_double::frees == frees + 1);
  return 0;
}

// Every large buffer of a second context of the same problem comes from the first one's.
int cache_holds_all() {
  igafd_ctx* c = setup(64, 3, nullptr, true);
  CHECK(c);
  igafd_destroy(c);
  hip_double::forget();
  c = setup(64, 3, nullptr, true);
  CHECK(c && hip_double::large_mallocs == 0);
  igafd_destroy(c);
  return 0;
}

// At most 8 GiB per device, the oldest given back first; blocks without use
// for 64 later requests are given back.
int cache_bound_and_age() {
  void* p[6];
  for (int d = 0; d < 2; ++d) {
    CHECK(hipSetDevice(d) == hipSuccess);
    for (void*& q : p) CHECK((q = take(2 * kGiB)) != nullptr);
    for (void* q : p) igafd::block_free(q);
    CHECK(hip_double::bytes_on(d) == 8 * kGiB);
    CHECK(hip_double::bytes_on(0) == 8 * kGiB);  // the other device's are its own
  }
  CHECK(hip_double::live.count(p[5]) == 1 && hip_double::live.count(p[2]) == 1);
  CHECK(hip_double::live.count(p[1]) == 0 && hip_double::live.count(p[0]) == 0);
  void* big = take(9 * kGiB);  // larger than the bound: never kept
  igafd::block_free(big);
  CHECK(hip_double::live.count(big) == 0);
  CHECK(igafd_release_cached() >= 0 && hip_double::bytes_on(0) == 0 && hip_double::bytes_on(1) == 0);
  void* old = take(32 * kMiB);
  igafd::block_free(old);
  for (int k = 0; k < 64; ++k) {
    void* q = take(2 * kMiB);
    CHECK(q && hip_double::live.count(old) == 1);
    igafd::block_free(q);
  }
  void* q = take(2 * kMiB);
  CHECK(q && hip_double::live.count(old) == 0);
  return 0;
}

// An allocation that fails is made again without the cached blocks, whatever it is for.
int cache_failed_allocation() {
  void* a = take(6 * kGiB);
  igafd::block_free(a);
  hip_double::capacity = 10 * kGiB;
  void* b = take(8 * kGiB);
  CHECK(b && hip_double::bytes_on(0) == 8 * kGiB);
  igafd::block_free(b);
  void* c = nullptr;
  CHECK(igafd::device_malloc(&c, 9 * kGiB) == hipSuccess && hip_double::bytes_on(0) == 9 * kGiB);
  CHECK(hipGetLastError() == hipSuccess);
  CHECK(!take(2 * kGiB));
  CHECK(std::string(igafd_last_error()).find("device allocation") != std::string::npos);
  CHECK(hipGetLastError() == hipSuccess);
  return 0;
}

// igafd_release_cached gives everything back that no context holds, and nothing else.
int cache_release() {
  igafd_ctx* live = setup(40, 3, nullptr, true);
  CHECK(live);
  const size_t held = hip_double::bytes_on(0);
  igafd_ctx* c = setup(40, 3, nullptr, true);
  CHECK(c);
  igafd_destroy(c);
  const size_t kept = hip_double::bytes_on(0) - held;
  CHECK(kept > 0 && kept <= 8 * kGiB);
  CHECK(igafd_release_cached() > 0);
  CHECK(hip_double::bytes_on(0) <= held);
  CHECK(igafd_release_cached() == 0);
  igafd_destroy(live);
  CHECK(igafd_release_cached() > 0);
  CHECK(hip_double::bytes_on(0) == 0 && hip_double::live.empty());
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int bad = 1;
  if (what == "destroy_waits") bad = destroy_waits();
  if (what == "destroyed_stream") bad = destroyed_stream();
  if (what == "eigen_budget") bad = eigen_budget();
  if (what == "host_memory") bad = host_memory();
  if (what == "lds_limits") bad = lds_limits();
  if (what == "adi_lines") bad = adi_lines();
  if (what == "adi_setup") bad = adi_setup();
  if (what == "tile_without_room") bad = tile_without_room();
  if (what == "device_memory") bad = device_memory();
  if (what == "cache_fit") bad = cache_fit();
  if (what == "cache_holds_all") bad = cache_holds_all();
  if (what == "cache_bound_and_age") bad = cache_bound_and_age();
  if (what == "cache_failed_allocation") bad = cache_failed_allocation();
  if (what == "cache_release") bad = cache_release();
  if (!bad) std::printf("OK\n");
  std::fflush(stdout);
  return bad;
}
