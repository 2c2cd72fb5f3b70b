// Contexts on the host runtime of hip_double.h.  The argument names a check;
// prints "OK" and returns 0 when it holds.
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "hip_double.h"
#include "igafd.h"

#define CHECK(x)                                             \
  do {                                                       \
    if (!(x)) {                                              \
      std::printf("FAILED line %d: %s\n", __LINE__, #x);     \
      return 1;                                              \
    }                                                        \
  } while (0)

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

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int bad = 1;
  if (what == "destroy_waits") bad = destroy_waits();
  if (what == "destroyed_stream") bad = destroyed_stream();
  if (!bad) std::printf("OK\n");
  std::fflush(stdout);
  return bad;
}
