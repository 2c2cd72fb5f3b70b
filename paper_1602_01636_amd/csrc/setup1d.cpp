// Host-side univariate setup: knot validation, Gauss-Legendre rule, B-spline
// values at the Gauss points, the 1D mass/stiffness matrices and their
// generalised eigendecomposition.
//
// Paper Sec. 2.1 (eq. knot-vector, eq. cox-deboor-1/2, eq. Vh), Sec. 3 (the
// univariate M_d, K_d) and Sec. 4.1 (generalised eigenproblem by Cholesky of M,
// symmetric eigendecomposition of L^-1 K L^-T, U = L^-T Ut).  The symmetric
// eigensolver is Householder tridiagonalisation plus implicit shifted QR.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <exception>
#include <thread>
#include <vector>

#include "internal.h"

namespace igafd {

// A team's threads spin at two barriers per reflector, so the decompositions
// that run at once share one budget of 16 team threads (or the CPUs, if fewer),
// by their work: share is one's part of it.  Setups on 16 CPUs with 16 for each
// and with 16 in all: n = 620-640 in three directions 152 and 129 ms, 700 x 1100
// 376 and 350 ms, 1000 x 1001 400 and 338 ms, 1500 x 1600 1.07 and 1.2 s (the same
// threads in equal shares: 700 x 1100 390 ms); one team at a time 260, 440, 510 ms
// and 1.4 s.
int eigen_threads(double share) {
  const int all = std::min(16, (int)std::thread::hardware_concurrency());
  return std::max(1, (int)(all * share));
}

namespace {

// Legendre polynomials P_q(z) and P_{q-1}(z) by the three-term recurrence.
void legendre(int q, double z, double* pq, double* pqm1) {
  double p0 = 1.0, p1 = z;
  for (int k = 2; k <= q; ++k) {
    const double pk = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
    p0 = p1;
    p1 = pk;
  }
  *pq = p1;
  *pqm1 = p0;
}

// Gauss-Legendre nodes and weights on [-1, 1]: Newton iteration on P_q with
// P_q'(z) = q (z P_q - P_{q-1}) / (z^2 - 1).
void gauss_legendre(int q, double* x, double* w) {
  for (int i = 0; i < q; ++i) {
    double z = std::cos(M_PI * (i + 0.75) / (q + 0.5));
    double pq = 0.0, pqm1 = 0.0;
    for (int it = 0; it < 100; ++it) {
      legendre(q, z, &pq, &pqm1);
      const double dz = pq / (q * (z * pq - pqm1) / (z * z - 1.0));
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    legendre(q, z, &pq, &pqm1);
    const double dp = q * (z * pq - pqm1) / (z * z - 1.0);
    x[q - 1 - i] = z;
    w[q - 1 - i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

// Values and first derivatives of the p+1 B-splines B_{k-p..k} that are
// nonzero on the span [t_k, t_{k+1}), at x in that span.  The degree is raised
// one step at a time with the two-term recursion (0/0 = 0); the derivative
// combines the degree p-1 values.
void span_basis(const double* t, int p, int k, double x, double* N, double* dN) {
  double cur[kMaxDegree + 2], nxt[kMaxDegree + 2], low[kMaxDegree + 2];
  cur[0] = 1.0;
  low[0] = 1.0;
  for (int j = 1; j <= p; ++j) {
    if (j == p)
      for (int i = 0; i < j; ++i) low[i] = cur[i];
    for (int i = 0; i <= j; ++i) {
      const int g = k - j + i;  // B_{g,j}
      double v = 0.0;
      if (i >= 1) {
        const double den = t[g + j] - t[g];
        if (den > 0.0) v += (x - t[g]) / den * cur[i - 1];
      }
      if (i <= j - 1) {
        const double den = t[g + j + 1] - t[g + 1];
        if (den > 0.0) v += (t[g + j + 1] - x) / den * cur[i];
      }
      nxt[i] = v;
    }
    for (int i = 0; i <= j; ++i) cur[i] = nxt[i];
  }
  for (int i = 0; i <= p; ++i) {
    N[i] = cur[i];
    const int g = k - p + i;
    double d = 0.0;
    if (i >= 1) {
      const double den = t[g + p] - t[g];
      if (den > 0.0) d += p / den * low[i - 1];
    }
    if (i <= p - 1) {
      const double den = t[g + p + 1] - t[g + 1];
      if (den > 0.0) d -= p / den * low[i];
    }
    dN[i] = d;
  }
}

// Runs fn(t, lo, hi) on `chunks` contiguous chunks t of [0, n), a host thread each;
// chunks whose thread cannot be started run on the caller's.  fn must not throw.
template <class F>
void parallel_rows(int n, int chunks, const F& fn) {
  auto chunk = [&](int t) { fn(t, (int)((long long)n * t / chunks), (int)((long long)n * (t + 1) / chunks)); };
  std::vector<std::thread> th;
  int t = 1;
  try {
    for (th.reserve(chunks); t < chunks; ++t) th.emplace_back(chunk, t);
  } catch (const std::exception&) {  // no thread, or no memory for one
  }
  chunk(0);
  for (; t < chunks; ++t) chunk(t);
  for (auto& x : th) x.join();
}

// Inner loops of the eigensolver over rows of doubles, compiled twice: for AVX2
// where the host has it, and for the baseline.  Every element is computed by
// the same operations in both (no FMA, no reordered sums), so the results do
// not depend on the host.
#define IGAFD_INLINE static inline __attribute__((always_inline))

// y += s x and y -= s x
IGAFD_INLINE void add_body(double* __restrict__ y, double s, const double* __restrict__ x, int n) {
  for (int j = 0; j < n; ++j) y[j] += s * x[j];
}
IGAFD_INLINE void sub_body(double* __restrict__ y, double s, const double* __restrict__ x, int n) {
  for (int j = 0; j < n; ++j) y[j] -= s * x[j];
}
// y -= a p + b v
IGAFD_INLINE void rank2_body(double* __restrict__ y, double a, const double* __restrict__ p, double b,
                             const double* __restrict__ v, int n) {
  for (int j = 0; j < n; ++j) y[j] -= a * p[j] + b * v[j];
}
// rotations q = 0..nrot-1 on the rows rk[q], rk[q] + 1 of T (rows of kRotRows values)
constexpr int kRotRows = 32;
IGAFD_INLINE void rotate_body(double* T, const int* rk, const double* rc, const double* rs, size_t nrot) {
  for (size_t q = 0; q < nrot; ++q) {
    double* __restrict__ a = T + (size_t)rk[q] * kRotRows;
    double* __restrict__ b = a + kRotRows;
    const double c = rc[q], s = rs[q];
    for (int j = 0; j < kRotRows; ++j) {
      const double va = a[j], vb = b[j];
      a[j] = c * va + s * vb;
      b[j] = -s * va + c * vb;
    }
  }
}

void add_base(double* y, double s, const double* x, int n) { add_body(y, s, x, n); }
void sub_base(double* y, double s, const double* x, int n) { sub_body(y, s, x, n); }
void rank2_base(double* y, double a, const double* p, double b, const double* v, int n) { rank2_body(y, a, p, b, v, n); }
void rotate_base(double* T, const int* rk, const double* rc, const double* rs, size_t n) { rotate_body(T, rk, rc, rs, n); }
#ifndef __HIP_DEVICE_COMPILE__  // host code only; the device pass of hipcc knows no x86 features
#define IGAFD_AVX2 __attribute__((target("avx2")))
IGAFD_AVX2 void add_avx2(double* y, double s, const double* x, int n) { add_body(y, s, x, n); }
IGAFD_AVX2 void sub_avx2(double* y, double s, const double* x, int n) { sub_body(y, s, x, n); }
IGAFD_AVX2 void rank2_avx2(double* y, double a, const double* p, double b, const double* v, int n) {
  rank2_body(y, a, p, b, v, n);
}
IGAFD_AVX2 void rotate_avx2(double* T, const int* rk, const double* rc, const double* rs, size_t n) {
  rotate_body(T, rk, rc, rs, n);
}
#endif

struct RowOps {
  void (*add)(double*, double, const double*, int) = add_base;
  void (*sub)(double*, double, const double*, int) = sub_base;
  void (*rank2)(double*, double, const double*, double, const double*, int) = rank2_base;
  void (*rotate)(double*, const int*, const double*, const double*, size_t) = rotate_base;
  RowOps() {
#ifndef __HIP_DEVICE_COMPILE__
    __builtin_cpu_init();
    if (__builtin_cpu_supports("avx2")) {
      add = add_avx2;
      sub = sub_avx2;
      rank2 = rank2_avx2;
      rotate = rotate_avx2;
    }
#endif
  }
};
const RowOps& ops() {
  static const RowOps o;
  return o;
}

// Largest |i - j| with A_ij != 0 (A n x n, row-major).
int bandwidth(const std::vector<double>& A, int n) {
  int bw = 0;
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < i; ++j)
      if (A[(size_t)i * n + j] != 0.0 || A[(size_t)j * n + i] != 0.0) {
        bw = std::max(bw, i - j);
        break;
      }
  return bw;
}

// Cholesky A = L L^T of a band matrix (bandwidth bw; lower factor in place,
// row-major, upper part zeroed).  The factor keeps the band.  False if not SPD.
bool cholesky(std::vector<double>& A, int n, int bw) {
  for (int j = 0; j < n; ++j) {
    double* aj = &A[(size_t)j * n];
    const int k0 = std::max(0, j - bw);
    double s = aj[j];
    for (int k = k0; k < j; ++k) s -= aj[k] * aj[k];
    if (!(s > 0.0)) return false;
    const double ljj = std::sqrt(s);
    aj[j] = ljj;
    for (int i = j + 1; i <= std::min(n - 1, j + bw); ++i) {
      double* ai = &A[(size_t)i * n];
      double v = ai[j];
      for (int k = std::max(k0, i - bw); k < j; ++k) v -= ai[k] * aj[k];
      ai[j] = v / ljj;
    }
    for (int k = j + 1; k < n; ++k) aj[k] = 0.0;
  }
  return true;
}

// X <- L^-1 X for a band lower factor L (forward substitution on whole rows).
void forward_rows(const std::vector<double>& L, int n, int bw, std::vector<double>& X) {
  for (int i = 0; i < n; ++i) {
    double* xi = &X[(size_t)i * n];
    for (int k = std::max(0, i - bw); k < i; ++k) {
      ops().sub(xi, L[(size_t)i * n + k], &X[(size_t)k * n], n);
    }
    const double d = L[(size_t)i * n + i];
    for (int j = 0; j < n; ++j) xi[j] /= d;
  }
}

// Symmetric eigensolver: Householder reduction to tridiagonal form followed by
// implicit QR steps with the Wilkinson shift (Golub & Van Loan, Sec. 8.3).
// S (n x n, row-major) is destroyed; on return lam holds the eigenvalues in
// ascending order and V the orthonormal eigenvectors as columns (V[i][k]).
// The QR steps run on the tridiagonal alone; their plane rotations are
// recorded and applied to V afterwards, a block of rows at a time.  The result
// does not depend on `team_max`, the most threads that meet at barriers.
void symmetric_eig(std::vector<double>& S, int n, std::vector<double>& lam, std::vector<double>& V, int team_max) {
  std::vector<double> Vt((size_t)n * n, 0.0);  // V transposed
  for (int i = 0; i < n; ++i) Vt[(size_t)i * n + i] = 1.0;
  std::vector<double> pv(n);
  const RowOps& op = ops();
  // 1. S = Q T Q^T: reflector k zeroes column k below the subdiagonal.  The
  // matrix-vector products run over rows (S is symmetric to the last bit: its
  // update is), each element summed in ascending order.  From kTeamMin on, a team
  // of threads runs the whole loop, each on a share of the columns (rows in the
  // update of S), with the scalars and v computed by every thread: below, the two
  // barriers per reflector cost more than they save (n = 515: 35 ms alone; a
  // thread started per product and reflector: 90).
  constexpr int kTeamMin = 600, kTeamCols = 96;
  const int team = n < kTeamMin ? 1 : std::max(1, std::min(team_max, n / kTeamCols));
  std::vector<double> mine((size_t)team * 3 * n);  // each thread's v, w, t: threads allocate nothing
  auto reflect = [&](int t, int T, auto&& barrier) {
    double *v = &mine[(size_t)t * 3 * n], *w = v + n, *tv = w + n;
    auto share = [&](int m, int* lo, int* hi) {
      *lo = (int)((long long)m * t / T);
      *hi = (int)((long long)m * (t + 1) / T);
    };
    int lo, hi;
    for (int k = 0; k + 2 < n; ++k) {
      const int m = n - k - 1;  // length of x = S[k+1:, k]
      const double* x = &S[(size_t)k * n + k + 1];
      double nx = 0.0;
      for (int i = 0; i < m; ++i) nx += x[i] * x[i];
      nx = std::sqrt(nx);
      if (nx == 0.0) continue;
      const double x0 = x[0];
      const double alpha = x0 >= 0 ? -nx : nx;
      for (int i = 0; i < m; ++i) v[i] = x[i];
      v[0] -= alpha;
      double nv = 0.0;
      for (int i = 0; i < m; ++i) nv += v[i] * v[i];
      nv = std::sqrt(nv);
      if (nv == 0.0) continue;
      for (int i = 0; i < m; ++i) v[i] /= nv;
      // trailing block B <- H B H = B - 2 v w^T - 2 w v^T, w = B v - (v^T B v) v
      share(m, &lo, &hi);
      for (int i = lo; i < hi; ++i) pv[i] = 0.0;
      for (int j = 0; j < m && lo < hi; ++j) op.add(&pv[lo], v[j], &S[(size_t)(k + 1 + j) * n + k + 1 + lo], hi - lo);
      barrier();
      double cvp = 0.0;
      for (int i = 0; i < m; ++i) cvp += v[i] * pv[i];
      for (int i = 0; i < m; ++i) w[i] = pv[i] - cvp * v[i];
      for (int i = lo; i < hi; ++i)
        op.rank2(&S[(size_t)(k + 1 + i) * n + k + 1], 2.0 * v[i], w, 2.0 * w[i], v, m);
      if (t == 0) {  // column and row k of S are read by nobody before the barrier
        S[(size_t)(k + 1) * n + k] = alpha;
        for (int i = 1; i < m; ++i) S[(size_t)(k + 1 + i) * n + k] = 0.0;
      }
      // V <- V H on columns k+1..n-1 (rows of V^T)
      share(n, &lo, &hi);
      for (int r = lo; r < hi; ++r) tv[r] = 0.0;
      for (int j = 0; j < m && lo < hi; ++j) op.add(&tv[lo], v[j], &Vt[(size_t)(k + 1 + j) * n + lo], hi - lo);
      for (int r = lo; r < hi; ++r) tv[r] *= 2.0;
      for (int j = 0; j < m && lo < hi; ++j) op.sub(&Vt[(size_t)(k + 1 + j) * n + lo], v[j], &tv[lo], hi - lo);
      barrier();
    }
  };
  if (team == 1) {
    reflect(0, 1, []() {});
  } else {
    std::atomic<int> arrived{0}, phase{0}, size{0};
    auto barrier = [&]() {
      const int ph = phase.load(std::memory_order_acquire);
      if (arrived.fetch_add(1, std::memory_order_acq_rel) + 1 == size.load(std::memory_order_relaxed)) {
        arrived.store(0, std::memory_order_relaxed);
        phase.store(ph + 1, std::memory_order_release);
      } else {
        for (int spin = 0; phase.load(std::memory_order_acquire) == ph; ++spin)
          if (spin > 2000) std::this_thread::yield();
      }
    };
    std::vector<std::thread> th;
    std::atomic<bool> go{false};
    try {
      th.reserve(team);
      for (int t = 1; t < team; ++t)
        th.emplace_back([&, t]() {
          while (!go.load(std::memory_order_acquire)) std::this_thread::yield();
          reflect(t, size.load(std::memory_order_relaxed), barrier);
        });
    } catch (const std::exception&) {  // fewer threads than asked for
    }
    size.store((int)th.size() + 1, std::memory_order_relaxed);
    go.store(true, std::memory_order_release);
    reflect(0, (int)th.size() + 1, barrier);
    for (auto& x : th) x.join();
  }
  std::vector<double> d(n), e(n, 0.0);
  for (int i = 0; i < n; ++i) d[i] = S[(size_t)i * n + i];
  for (int i = 0; i + 1 < n; ++i) e[i] = S[(size_t)(i + 1) * n + i];
  // 2. implicit QR steps on unreduced blocks [lo, hi] of the tridiagonal T;
  // rotation j acts on columns (rk[j], rk[j] + 1) of V
  std::vector<int> rk;
  std::vector<double> rc, rs;
  const double eps = 2.2e-16;
  int hi = n - 1, guard = 0;
  while (hi > 0 && guard < 100 * n) {
    if (std::fabs(e[hi - 1]) <= eps * (std::fabs(d[hi - 1]) + std::fabs(d[hi]))) {
      e[hi - 1] = 0.0;
      --hi;
      continue;
    }
    ++guard;
    int lo = hi - 1;
    while (lo > 0 && std::fabs(e[lo - 1]) > eps * (std::fabs(d[lo - 1]) + std::fabs(d[lo]))) --lo;
    // Wilkinson shift: eigenvalue of the trailing 2x2 closer to d[hi]
    const double delta = 0.5 * (d[hi - 1] - d[hi]);
    const double eh = e[hi - 1];
    const double den = delta + (delta >= 0 ? 1.0 : -1.0) * std::sqrt(delta * delta + eh * eh);
    const double mu = d[hi] - eh * eh / den;
    double x = d[lo] - mu, z = e[lo];
    for (int k = lo; k < hi; ++k) {
      // rotation in the (k, k+1) plane taking (x, z) to (r, 0)
      const double r = std::hypot(x, z);
      const double c = r == 0.0 ? 1.0 : x / r, s = r == 0.0 ? 0.0 : z / r;
      if (k > lo) e[k - 1] = r;  // (x, z) were (e[k-1], bulge)
      const double a = d[k], b = e[k], cc = d[k + 1];
      d[k] = c * c * a + 2.0 * c * s * b + s * s * cc;
      d[k + 1] = s * s * a - 2.0 * c * s * b + c * c * cc;
      e[k] = c * s * (cc - a) + (c * c - s * s) * b;
      if (k + 1 < hi) {
        const double next = e[k + 1];
        x = e[k];
        z = s * next;        // new bulge at (k, k+2)
        e[k + 1] = c * next;
      }
      rk.push_back(k);
      rc.push_back(c);
      rs.push_back(s);
    }
  }
  // 3. V <- V G_1 G_2 ...: blocks of rows of V, stored transposed so that one
  // rotation updates two contiguous runs
  V.assign((size_t)n * n, 0.0);
  constexpr int B = kRotRows;
  const size_t nrot = rk.size();
  const int blocks = (n + B - 1) / B, chunks = n < 256 ? 1 : std::min(eigen_threads(1.0), blocks);
  std::vector<double> runs((size_t)chunks * n * B);
  parallel_rows(blocks, chunks, [&](int t, int blo, int bhi) {
    double* T = &runs[(size_t)t * n * B];
    for (int blk = blo; blk < bhi; ++blk) {
      const int r0 = blk * B, nb = std::min(B, n - r0);
      for (int k = 0; k < n; ++k)
        for (int j = 0; j < nb; ++j) T[(size_t)k * B + j] = Vt[(size_t)k * n + r0 + j];
      op.rotate(T, rk.data(), rc.data(), rs.data(), nrot);
      for (int j = 0; j < nb; ++j)
        for (int k = 0; k < n; ++k) V[(size_t)(r0 + j) * n + k] = T[(size_t)k * B + j];
    }
  });
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::sort(order.begin(), order.end(), [&](int a, int b) { return d[a] < d[b]; });
  lam.resize(n);
  std::vector<double> Vs((size_t)n * n);
  for (int k = 0; k < n; ++k) {
    lam[k] = d[order[k]];
    for (int i = 0; i < n; ++i) Vs[(size_t)i * n + k] = V[(size_t)i * n + order[k]];
  }
  V.swap(Vs);
}

}  // namespace

igafd_status build_direction(int p, int q, int nknots, const double* knots, Dir1D* out, bool eig) {
  if (p < 1 || p > kMaxDegree) {
    set_error("degree must be in 1.." + std::to_string(kMaxDegree));
    return IGAFD_ERR_ARG;
  }
  if (q != p + 1) {
    set_error("the library integrates with p+1 Gauss points per element and direction");
    return IGAFD_ERR_ARG;
  }
  if (!knots || nknots < 2 * p + 2) {
    set_error("knot vector too short for the degree");
    return IGAFD_ERR_ARG;
  }
  const double* t = knots;
  for (int i = 0; i + 1 < nknots; ++i)
    if (!(t[i] <= t[i + 1])) {
      set_error("knots must be nondecreasing");
      return IGAFD_ERR_ARG;
    }
  for (int i = 0; i <= p; ++i)
    if (t[i] != 0.0 || t[nknots - 1 - i] != 1.0) {
      set_error("knot vector must be open on [0,1]");
      return IGAFD_ERR_ARG;
    }
  if (t[p + 1] == 0.0 || t[nknots - p - 2] == 1.0) {
    set_error("end knots repeated more than p+1 times");
    return IGAFD_ERR_ARG;
  }
  for (int i = p + 1; i < nknots - p - 1;) {
    int j = i;
    while (j < nknots - p - 1 && t[j] == t[i]) ++j;
    if (j - i > p) {
      set_error("interior knot multiplicity exceeds p");
      return IGAFD_ERR_ARG;
    }
    i = j;
  }
  Dir1D& d = *out;
  d.p = p;
  d.q = q;
  d.knots.assign(t, t + nknots);
  d.m = nknots - p - 1;
  d.n = d.m - 2;
  if (d.n < 1) {
    set_error("no interior basis functions");
    return IGAFD_ERR_ARG;
  }
  std::vector<double> gx(q), gw(q);
  gauss_legendre(q, gx.data(), gw.data());
  d.elem_first.clear();
  d.qx.clear();
  d.qw.clear();
  d.val.clear();
  d.der.clear();
  for (int k = p; k < d.m; ++k) {
    if (!(t[k] < t[k + 1])) continue;
    d.elem_first.push_back(k - p);
    const double a = t[k], b = t[k + 1];
    for (int s = 0; s < q; ++s) {
      const double x = a + 0.5 * (b - a) * (gx[s] + 1.0);
      d.qx.push_back(x);
      d.qw.push_back(0.5 * (b - a) * gw[s]);
      double N[kMaxDegree + 1], dN[kMaxDegree + 1];
      span_basis(t, p, k, x, N, dN);
      for (int i = 0; i <= p; ++i) {
        d.val.push_back(N[i]);
        d.der.push_back(dN[i]);
      }
    }
  }
  d.nel = (int)d.elem_first.size();
  const int n = d.n;
  d.M.assign((size_t)n * n, 0.0);
  d.K.assign((size_t)n * n, 0.0);
  for (int e = 0; e < d.nel; ++e) {
    for (int s = 0; s < q; ++s) {
      const double w = d.qw[e * q + s];
      const double* v = &d.val[(e * q + s) * (p + 1)];
      const double* dv = &d.der[(e * q + s) * (p + 1)];
      for (int a = 0; a <= p; ++a) {
        const int ia = d.elem_first[e] + a - 1;
        if (ia < 0 || ia >= n) continue;
        for (int b = 0; b <= p; ++b) {
          const int ib = d.elem_first[e] + b - 1;
          if (ib < 0 || ib >= n) continue;
          d.M[ia * n + ib] += w * v[a] * v[b];
          d.K[ia * n + ib] += w * dv[a] * dv[b];
        }
      }
    }
  }
  d.U.clear();
  d.lam.clear();
  return eig ? eigen_direction(out, eigen_threads(1.0)) : IGAFD_OK;
}

igafd_status eigen_direction(Dir1D* out, int team_max) {
  Dir1D& d = *out;
  const int n = d.n;
  // generalised eigendecomposition K U = M U D, U^T M U = I
  const int bw = bandwidth(d.M, n);
  std::vector<double> L = d.M;
  if (!cholesky(L, n, bw)) {
    set_error("Cholesky of the 1D mass matrix failed");
    return IGAFD_ERR_NOT_SPD;
  }
  // S = L^-1 K L^-T = L^-1 (L^-1 K)^T (K symmetric)
  std::vector<double> X = d.K;
  forward_rows(L, n, bw, X);
  std::vector<double> S((size_t)n * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) S[(size_t)j * n + i] = X[(size_t)i * n + j];
  forward_rows(L, n, bw, S);
  for (int i = 0; i < n; ++i)
    for (int j = i + 1; j < n; ++j) {
      const double s = 0.5 * (S[(size_t)i * n + j] + S[(size_t)j * n + i]);
      S[(size_t)i * n + j] = S[(size_t)j * n + i] = s;
    }
  std::vector<double> Ut;
  symmetric_eig(S, n, d.lam, Ut, team_max);
  // U = L^-T Ut: backward substitution on whole rows, L^T upper with band bw
  d.U = Ut;
  for (int i = n - 1; i >= 0; --i) {
    double* ui = &d.U[(size_t)i * n];
    for (int k = i + 1; k <= std::min(n - 1, i + bw); ++k) {
      ops().sub(ui, L[(size_t)k * n + i], &d.U[(size_t)k * n], n);
    }
    const double dd = L[(size_t)i * n + i];
    for (int j = 0; j < n; ++j) ui[j] /= dd;
  }
  return IGAFD_OK;
}

}  // namespace igafd
