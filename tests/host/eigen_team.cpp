// The eigensolver's thread team, host only: from 600 unknowns on one
// decomposition runs on several threads that meet at barriers, and several
// decompositions run at once.  Eigenvalues and vectors must be those of one
// thread bit for bit, for team sizes that do and do not divide the rows, alone
// and side by side.  With an argument, only two decompositions of that
// many unknowns side by side (for a build with the thread sanitizer).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <thread>
#include <vector>

#include "internal.h"

namespace igafd {
void set_error(const std::string&) {}
}  // namespace igafd

namespace {

igafd::Dir1D direction(int n, int p, double bend) {  // n = E + p - 2 unknowns, graded knots
  const int E = n + 2 - p;
  std::vector<double> k(p + 1, 0.0);
  for (int e = 1; e < E; ++e) {
    const double x = (double)e / E;
    k.push_back(x + bend * x * (1.0 - x));
  }
  k.insert(k.end(), p + 1, 1.0);
  igafd::Dir1D d;
  if (igafd::build_direction(p, p + 1, (int)k.size(), k.data(), &d, false) != IGAFD_OK) std::abort();
  return d;
}

igafd::Dir1D solved(const igafd::Dir1D& d, int threads) {
  igafd::Dir1D r = d;
  if (igafd::eigen_direction(&r, threads) != IGAFD_OK) std::abort();
  return r;
}

}  // namespace

int main(int argc, char** argv) {
  const int n0 = argc > 1 ? std::atoi(argv[1]) : 599;
  const bool all = argc < 2;
  int bad = 0;
  std::vector<igafd::Dir1D> dirs, ref;
  for (int k = 0; k < (all ? 3 : 2); ++k) {
    dirs.push_back(direction(n0 + (k == 2 ? 73 : k), 2 + k, 0.2 * k));
    if (all) ref.push_back(solved(dirs.back(), 1));
  }
  auto same = [&](const igafd::Dir1D& d, size_t k, const char* what, int threads) {
    if (!all || d.U == ref[k].U && d.lam == ref[k].lam) return;
    std::printf("FAILED: n = %d on %d threads (%s) differs from one thread\n", d.n, threads, what);
    ++bad;
  };
  for (int threads : {2, 3, 5, 16})
    for (size_t k = 0; k < dirs.size() && all; ++k) same(solved(dirs[k], threads), k, "alone", threads);
  const int threads = igafd::eigen_threads(1.0 / (double)dirs.size());
  if (threads < 1 || threads * (int)dirs.size() > std::max(16, (int)dirs.size())) ++bad;
  std::vector<igafd::Dir1D> got(dirs);
  std::vector<std::thread> th;
  for (size_t k = 0; k < dirs.size(); ++k) th.emplace_back([&, k]() { got[k] = solved(dirs[k], 2); });
  for (std::thread& t : th) t.join();
  for (size_t k = 0; k < dirs.size(); ++k) same(got[k], k, "side by side", 2);
  std::printf("%s\n", bad ? "FAILED" : "OK");
  return bad ? 1 : 0;
}
