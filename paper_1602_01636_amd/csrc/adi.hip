// Three-variable ADI of Douglas as an inexact application of P^-1
// (Sec. 5.2 eq. ADI3D, eq. ADI3D2, Alg. "3D ADI method"; used inside CG as
// the preconditioner P_J of Sec. 4.2 Thm. ADIprec, which keeps it SPD).
//
// Parameters: [a, b] spans the eigenvalues of M_d^-1 K_d over the three
// directions; for a count J the parameters are geometric between a and b,
// omega_j = a (b/a)^((j-1)/(J-1)); J is the smallest count whose error
// operator has ||T_J|| <= eps, at most J0 = ceil(1.16 ln(b/a) ln(1/eps))
// (eq. ADI3Diter).  T_J is diagonal in the eigenvector basis of the three
// pencils with entries prod_j g_j(l1, l2, l3),
//   g_j = 1 - 2 omega_j^2 (l1 + l2 + l3) / ((omega_j + l1)(omega_j + l2)(omega_j + l3)),
// so ||T_J|| is evaluated exactly as the largest |prod_j g_j| over the
// triples of eigenvalues (host, at setup).
//
// Device: a step is four sub-steps along one direction each, fused in LDS (k_adi)
// for lines whose tiles fit; along longer lines a sub-step is a banded product
// (one thread per grid point) and a banded Cholesky solve (one thread per grid
// line, walking it in chunks: the next chunk's values load while the recurrence
// runs on the current one in registers with a window of p values).  Lines of
// directions 2 and 3 are taken by consecutive threads at consecutive i1, so their
// loads are coalesced.
#include <algorithm>
#include <cmath>
#include <memory>
#include <thread>
#include <vector>

#include "internal.h"
#include "reduce.h"

namespace igafd {
namespace {

// Lines of direction DIR: count, start offset and stride in the (n3, n2, n1) grid.
template <int DIR>
__device__ inline bool line_of(long long l, int n1, int n2, int n3, long long* base, long long* stride, int* len) {
  if (DIR == 0) {
    if (l >= (long long)n2 * n3) return false;
    *base = l * n1;
    *stride = 1;
    *len = n1;
  } else if (DIR == 1) {
    if (l >= (long long)n1 * n3) return false;
    const long long i3 = l / n1, i1 = l % n1;
    *base = i3 * n1 * n2 + i1;
    *stride = n1;
    *len = n2;
  } else {
    if (l >= (long long)n1 * n2) return false;
    *base = l;
    *stride = (long long)n1 * n2;
    *len = n3;
  }
  return true;
}

// rows of the bands and of the fused sub-steps' factors: padded to whole 16-byte reads
constexpr int even_up(int n) { return (n + 1) & ~1; }
constexpr int kLineBlock = 64;  // threads per block of the line solves (few lines: spread over CUs)
constexpr int kChunk = 16;      // line values loaded together in the solves

// y = cz z + ca B (x + c2 x2) along direction DIR, B a band [n][even_up(2P+1)]: one
// thread per grid point (the neighbours along DIR are other threads' points,
// read through the caches).  z may be y; x and x2 may not.
template <int P, int DIR>
__global__ __launch_bounds__(kBlock) void k_band_apply(const double* __restrict__ Bd, double ca,
                                                      const double* __restrict__ x, const double* __restrict__ x2,
                                                      double c2, const double* z, double cz, double* y, int n1, int n2,
                                                      int n3, const int* __restrict__ flag) {
  if (flag && *flag) return;
  const long long N = (long long)n1 * n2 * n3;
  const long long o = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (o >= N) return;
  int i, len;
  long long stride;
  if (DIR == 0) {
    i = (int)(o % n1);
    len = n1;
    stride = 1;
  } else if (DIR == 1) {
    i = (int)((o / n1) % n2);
    len = n2;
    stride = n1;
  } else {
    i = (int)(o / ((long long)n1 * n2));
    len = n3;
    stride = (long long)n1 * n2;
  }
  constexpr int W = 2 * P + 1, WP = even_up(W);
  double acc = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const int j = i + k - P;
    if (j >= 0 && j < len) {
      const long long q = o + (long long)(k - P) * stride;
      const double w = x2 ? x[q] + c2 * x2[q] : x[q];
      acc = fma(Bd[(long long)i * WP + k], w, acc);
    }
  }
  y[o] = (z ? cz * z[o] : 0.0) + ca * acc;
}

// y = (L L^T)^-1 (alpha x) along direction DIR; L lower band [len][P+1] with
// L[i][k] = L_{i, i-k} for k >= 1 and L[i][0] = 1 / L_{i,i}.  One thread per
// line.  The factor (the same for every line) is staged in LDS first, so the
// recurrence reads its coefficients from LDS, not memory; the line is read in
// chunks of kChunk values, the next chunk's loads issued before the current
// chunk's recurrence.  len is the (uniform) line length.  In place (x == y)
// allowed: a chunk is loaded before any of its values is written, and writes
// never reach a chunk that is still to be loaded.
template <int P, int DIR>
__global__ __launch_bounds__(kLineBlock) void k_line_solve(const double* __restrict__ L, double alpha, const double* x,
                                                          double* y, int n1, int n2, int n3, int len,
                                                          const int* __restrict__ flag) {
  if (flag && *flag) return;
  extern __shared__ double Ls[];  // [len][P+1]
  constexpr int W = P + 1;
  for (int e = threadIdx.x; e < len * W; e += kLineBlock) Ls[e] = L[e];
  __syncthreads();
  long long base, stride;
  int len_t;
  if (!line_of<DIR>((long long)blockIdx.x * kLineBlock + threadIdx.x, n1, n2, n3, &base, &stride, &len_t)) return;
  const int nch = (len + kChunk - 1) / kChunk;
  auto ld = [&](const double* src, int i0, double (&b)[kChunk]) {
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      const int i = i0 + c < len ? i0 + c : len - 1;
      b[c] = src[base + (long long)i * stride];
    }
  };
  auto st = [&](int i0, const double (&b)[kChunk]) {
#pragma unroll
    for (int c = 0; c < kChunk; ++c)
      if (i0 + c < len) y[base + (long long)(i0 + c) * stride] = b[c];
  };
  double win[P > 0 ? P : 1];  // the last P values (most recent last)
  double cur[kChunk], nxt[kChunk];
#pragma unroll
  for (int k = 0; k < P; ++k) win[k] = 0.0;
  ld(x, 0, cur);
  for (int q = 0; q < nch; ++q) {  // forward: L t = alpha x
    const int i0 = q * kChunk;
    if (q + 1 < nch) ld(x, i0 + kChunk, nxt);
#pragma unroll
    for (int c = 0; c < kChunk; ++c) {
      const int i = i0 + c;
      if (i < len) {
        double t = alpha * cur[c];
#pragma unroll
        for (int k = 1; k <= P; ++k) t -= Ls[i * W + k] * win[P - k];
        t *= Ls[i * W];
        cur[c] = t;
#pragma unroll
        for (int k = 0; k + 1 < P; ++k) win[k] = win[k + 1];
        if (P > 0) win[P - 1] = t;
      }
    }
    st(i0, cur);
#pragma unroll
    for (int c = 0; c < kChunk; ++c) cur[c] = nxt[c];
  }
#pragma unroll
  for (int k = 0; k < P; ++k) win[k] = 0.0;
  ld(y, (nch - 1) * kChunk, cur);
  for (int q = nch - 1; q >= 0; --q) {  // backward: L^T z = t, chunks from the end
    const int i0 = q * kChunk;
    if (q > 0) ld(y, i0 - kChunk, nxt);
#pragma unroll
    for (int c = kChunk - 1; c >= 0; --c) {
      const int i = i0 + c;
      if (i < len) {
        double zv = cur[c];
#pragma unroll
        for (int k = 1; k <= P; ++k)
          if (i + k < len) zv -= Ls[(i + k) * W + k] * win[P - k];
        zv *= Ls[i * W];
        cur[c] = zv;
#pragma unroll
        for (int k = 0; k + 1 < P; ++k) win[k] = win[k + 1];
        if (P > 0) win[P - 1] = zv;
      }
    }
    st(i0, cur);
#pragma unroll
    for (int c = 0; c < kChunk; ++c) cur[c] = nxt[c];
  }
}

// ---- fused sub-steps ----
// A Douglas step is four sub-steps, each along one direction: combine vectors,
// one or two banded products, one banded Cholesky solve.  A block takes LT lines
// through all of it in LDS (tiles [i][line], rows padded to LT + 1), so a
// sub-step reads each of its vectors once and writes its results once:
//   A (dir 2): u = M2^-1 K2 s                                    2 passes
//   B (dir 1): s* = (K1 + w M1)^-1 (r~ - (K1 - w M1) s - 2 M1 (u + v))   5
//   C (dir 2): s** = (K2 + w M2)^-1 M2 (u + w s*)                 3
//   D (dir 3): b = v + w s**; s = (K3 + w M3)^-1 M3 b; v = b - w s      4
// Bound by latency: loads, product, two sweeps of a dependent chain over the line
// and stores follow each other in a block, and 32 lines a block spread 97^2 lines
// over all CUs once.  Measured at 97^3, p = 3 (launches that run; those behind the
// stop flag end in 3 us): sub-steps A to D 17, 22, 18 and 20 us (about 7 of it for
// moving the vectors, 2 for the tables, 2 for the product, 6 for the sweeps, about
// 170 clocks per 4 rows each way), a step 78 us; the same step as ten launches
// (five products, four solves, an update: 35 passes) took 247 us, most of it in solves
// whose lines were loaded one value at a time.  Without the push form of the sweep
// (four dependent multiply-adds a row, loads next to their use) a sub-step took 18
// to 32 us; every load of a block in flight before the first wait did not pay (+1 us).
enum { ADI_INIT = 0, ADI_A = 1, ADI_B = 2, ADI_C = 3, ADI_D = 4 };
constexpr int kAdiThreads = 256;
constexpr size_t kAdiLds = 160 * 1024 - 64;  // less the block sum

struct AdiArgs {
  const double *x0, *x1, *x2, *x3;  // inputs of the sub-step
  const double *band0, *band1;      // bands of its products
  double *y0, *y1;
  double c;                         // w, or the factor of the right-hand side (INIT)
  int first;                        // s, u and v are zero
  int n1, n2, n3;
  double* partial;                  // D: block sums of x2 . y0 (x2 = r), or null
  const int* flag;
};

constexpr int kAdiU = 4;  // rows a sweep loads together
constexpr int adi_tiles(int mode) { return mode == ADI_B || mode == ADI_D ? 2 : 1; }
constexpr int adi_bands(int mode) { return mode == ADI_INIT ? 0 : mode == ADI_B ? 2 : 1; }
// rows of a sweep: whole turns of its loop
constexpr int adi_rows(int len) { return (len + 2 * kAdiU - 1) / (2 * kAdiU) * (2 * kAdiU); }
template <int P>
size_t adi_lds(int mode, int lt, int len) {
  return sizeof(double) * ((size_t)2 * adi_rows(len) * even_up(P + 1) +
                           (size_t)len * (adi_bands(mode) * even_up(2 * P + 1) + (adi_tiles(mode) - 1) * (lt + 1)) +
                           (size_t)(adi_rows(len) + 2 * P) * (lt + 1));
}

// One sweep of a line's solve on its LDS column (lane = line): column rows
// r0 + m dr, m = 0 .. rows-1 (a whole number of turns; the rows beyond the line are
// zeros), hold d_m b_m and become z_m = d_m b_m - sum_k g_{m-k,k} z_{m-k} (times
// d_m if SCALE: what the sweep back starts from).  f: [rows][RP] = d_m, g_m1 .. g_mP
// in sweep order.  A value is pushed into the P rows after it, so a row waits for
// one multiply-add only.  The next U rows load while U rows are worked on (two
// register sets, no moves between them); up to P rows past the sweep are read.
template <int P, bool SCALE>
__device__ inline void adi_sweep(const double* __restrict__ f, double* col, int dr, int rows) {
  constexpr int U = kAdiU, RP = even_up(P + 1);
  double pend[P];  // rows m .. m+P-1 less what is known of their sums
#pragma unroll
  for (int d = 0; d < P; ++d) pend[d] = col[d * dr];
  auto load = [&](int m0, double (&w)[U][RP], double (&x)[U]) {
    const int m = m0 < rows ? m0 : 0;  // past the end: any rows, not used
#pragma unroll
    for (int k = 0; k < U; ++k) {
#pragma unroll
      for (int d = 0; d < RP; d += 2) {
        const double2 v = *reinterpret_cast<const double2*>(f + (m + k) * RP + d);
        w[k][d] = v.x;
        w[k][d + 1] = v.y;
      }
      x[k] = col[(m + k + P) * dr];
    }
  };
  auto run = [&](int m0, const double (&w)[U][RP], const double (&x)[U]) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const double z = pend[0];
#pragma unroll
      for (int d = 1; d <= P; ++d) pend[d - 1] = fma(-w[k][d], z, d < P ? pend[d] : x[k]);
      col[(m0 + k) * dr] = SCALE ? w[k][0] * z : z;
    }
  };
  double wa[U][RP], wb[U][RP], xa[U], xb[U];
  load(0, wa, xa);
  for (int m0 = 0; m0 < rows; m0 += 2 * U) {
    load(m0 + U, wb, xb);
    __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of the rows that run meanwhile
    run(m0, wa, xa);
    __builtin_amdgcn_sched_barrier(0);
    load(m0 + 2 * U, wa, xa);
    __builtin_amdgcn_sched_barrier(0);
    run(m0 + U, wb, xb);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int P, int DIR, int LT, int MODE>
__global__ __launch_bounds__(kAdiThreads) void k_adi(AdiArgs a, const double* __restrict__ fac) {
  if (a.flag && *a.flag) return;
  extern __shared__ __attribute__((aligned(16))) double sm[];
  constexpr int TS = LT + 1, W = 2 * P + 1, WP = even_up(W), RP = even_up(P + 1), RG = kAdiThreads / LT, U = 16;
  const int len = DIR == 0 ? a.n1 : DIR == 1 ? a.n2 : a.n3;
  const int rows = adi_rows(len);
  const int tid = threadIdx.x;
  double* F = sm;  // forward, then backward rows
  double* B0 = F + 2 * rows * RP;
  double* Y = B0 + adi_bands(MODE) * len * WP + P * TS;  // P rows before and after it are read, not used
  double* X = Y + (rows + P) * TS;                       // B: u + v; D: b
  const long long nlines = DIR == 0 ? (long long)a.n2 * a.n3 : DIR == 1 ? (long long)a.n1 * a.n3 : (long long)a.n1 * a.n2;
  const long long l0 = (long long)blockIdx.x * LT;
  const int nl = (int)(nlines - l0 < LT ? nlines - l0 : LT);
  // element (i, t): directions 2 and 3: thread t = tid % LT, rows i = tid / LT + k RG; direction 1: contiguous
  const int t = tid % LT, rg = tid / LT;
  long long base = 0, stride = 0;
  int len_t = 0;
  if (DIR != 0) (void)line_of<DIR>(l0 + (t < nl ? t : 0), a.n1, a.n2, a.n3, &base, &stride, &len_t);
  const int count = DIR == 0 ? nl * len : t < nl ? len : 0;
  const int start = DIR == 0 ? tid : rg, step = DIR == 0 ? kAdiThreads : RG;
  const int sq = DIR == 0 ? kAdiThreads / len : 0, sr = DIR == 0 ? kAdiThreads % len : 0;
  // the elements of the block's lines, U at a time: get(q, v) loads from global
  // offset q, put(i, slot, q, v) uses the values for row i at a tile slot
  auto at = [&](int e) { return DIR == 0 ? l0 * len + e : base + (long long)e * stride; };
  auto fetch = [&](int e0, auto&& get, double (&v)[U][3]) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int e = e0 + k * step;
      get(at(e < count ? e : 0), v[k]);
    }
  };
  auto spread = [&](int e0, int& ii, int& tt, auto&& put, const double (&v)[U][3]) {
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int e = e0 + k * step;
      const int i = DIR == 0 ? ii : e;
      if (e < count) put(i, i * TS + (DIR == 0 ? tt : t), at(e), v[k]);
      if (DIR == 0) {
        tt += sq;
        ii += sr;
        if (ii >= len) {
          ii -= len;
          tt += 1;
        }
      }
    }
  };
  auto each = [&](auto&& get, auto&& put) {
    int ii = DIR == 0 ? tid % len : 0, tt = DIR == 0 ? tid / len : 0;
    for (int e0 = start; e0 < count; e0 += U * step) {
      double v[U][3];
      fetch(e0, get, v);
      spread(e0, ii, tt, put, v);
    }
  };
  for (int k = tid; k < 2 * rows * RP; k += kAdiThreads) F[k] = fac[k];
  for (int k = tid; MODE != ADI_INIT && k < len * WP; k += kAdiThreads) {
    B0[k] = a.band0[k];
    if (MODE == ADI_B) B0[len * WP + k] = a.band1[k];
  }
  for (int k = tid; k < (rows - len) * TS; k += kAdiThreads) Y[len * TS + k] = 0.0;
  if (MODE == ADI_INIT) {
    __syncthreads();
    each([&](long long q, double* v) { v[0] = a.x0[q]; },
         [&](int i, int s, long long, const double* v) { Y[s] = F[i * RP] * (a.c * v[0]); });
  }
  if (MODE == ADI_A)
    each([&](long long q, double* v) { v[0] = a.x0[q]; },
         [&](int, int s, long long, const double* v) { Y[s] = v[0]; });
  if (MODE == ADI_B && !a.first)
    each(
        [&](long long q, double* v) {
          v[0] = a.x0[q];
          v[1] = a.x1[q];
          v[2] = a.x2[q];
        },
        [&](int, int s, long long, const double* v) {
          Y[s] = v[0];
          X[s] = v[1] + v[2];
        });
  if (MODE == ADI_C || MODE == ADI_D)
    each(
        [&](long long q, double* v) {
          v[0] = a.first ? 0.0 : a.x0[q];
          v[1] = a.x1[q];
        },
        [&](int, int s, long long, const double* v) { (MODE == ADI_D ? X : Y)[s] = v[0] + a.c * v[1]; });
  __syncthreads();
  // banded products into Y: thread (t, rg) takes a run of rows of line t, its
  // neighbours in a register window (rows outside the line have zero band
  // entries).  Y in place (A, B, C): the neighbouring runs' rows are read before any write.
  if (MODE != ADI_INIT && !(MODE == ADI_B && a.first)) {
    const int most = (len + RG - 1) / RG, per = most < P ? P : most;
    const int i0 = rg * per, i1 = i0 + per < len ? i0 + per : len;
    const bool work = t < nl && i0 < len;
    double* src = MODE == ADI_D ? X : Y;
    double x[W], hx[P], x2[W], hx2[P];
    if (work) {
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const int lo = i0 + k - P > 0 ? i0 + k - P : 0, hi = i1 + k < len ? i1 + k : len - 1;
        x[k + 1] = src[lo * TS + t];
        hx[k] = src[hi * TS + t];
        if (MODE == ADI_B) {
          x2[k + 1] = X[lo * TS + t];
          hx2[k] = X[hi * TS + t];
        }
      }
    }
    if (MODE != ADI_D) __syncthreads();
    if (work) {
#pragma unroll
      for (int k = 0; k < P; ++k) {  // rows i0 .. i0+P-1, or past a short last run: its halo
        const int i = i0 + k < len ? i0 + k : len - 1;
        x[P + 1 + k] = src[i * TS + t];
        if (MODE == ADI_B) x2[P + 1 + k] = X[i * TS + t];
      }
      auto row = [&](int i, double xn, double x2n) {
#pragma unroll
        for (int k = 0; k < W - 1; ++k) {
          x[k] = x[k + 1];
          if (MODE == ADI_B) x2[k] = x2[k + 1];
        }
        x[W - 1] = xn;
        if (MODE == ADI_B) x2[W - 1] = x2n;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int k = 0; k < WP; k += 2) {
          const double2 v = *reinterpret_cast<const double2*>(B0 + i * WP + k);
          s0 = fma(v.x, x[k], s0);
          if (k + 1 < W) s0 = fma(v.y, x[k + 1], s0);
          if (MODE == ADI_B) {
            const double2 u = *reinterpret_cast<const double2*>(B0 + (len + i) * WP + k);
            s1 = fma(u.x, x2[k], s1);
            if (k + 1 < W) s1 = fma(u.y, x2[k + 1], s1);
          }
        }
        Y[i * TS + t] = MODE == ADI_B ? -s0 - 2.0 * s1 : F[i * RP] * s0;
      };
      int i = i0;
      for (; i + P < i1; ++i) row(i, src[(i + P) * TS + t], MODE == ADI_B ? X[(i + P) * TS + t] : 0.0);
#pragma unroll
      for (int k = 0; k < P; ++k)  // the run's last P rows
        if (i1 - P + k >= i0) row(i1 - P + k, hx[k], MODE == ADI_B ? hx2[k] : 0.0);
    }
  }
  if (MODE == ADI_B) {
    __syncthreads();
    each([&](long long q, double* v) { v[0] = a.x3[q]; },
         [&](int i, int s, long long, const double* v) { Y[s] = F[i * RP] * (a.first ? v[0] : v[0] + Y[s]); });
  }
  __syncthreads();
  if (tid < nl) {
    adi_sweep<P, true>(F, Y + tid, TS, rows);
    adi_sweep<P, false>(F + rows * RP, Y + (rows - 1) * TS + tid, -TS, rows);
  }
  __syncthreads();
  double dot = 0.0;
  each(
      [&](long long q, double* v) {
        if (MODE == ADI_D && a.partial) v[0] = a.x2[q];
      },
      [&](int, int s, long long q, const double* v) {
        a.y0[q] = Y[s];
        if (MODE == ADI_D) {
          a.y1[q] = X[s] - a.c * Y[s];
          if (a.partial) dot = fma(v[0], Y[s], dot);
        }
      });
  if (MODE == ADI_D && a.partial) {
    const double sum = block_sum(dot);
    if (tid == 0) a.partial[blockIdx.x] = sum;
  }
}

__global__ void k_adi_fill0(double* __restrict__ a, double* __restrict__ b, long long N, const int* __restrict__ flag) {
  if (flag && *flag) return;
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (i < N) {
    a[i] = 0.0;
    b[i] = 0.0;
  }
}

// v = v + omega (s2 - s); with partial: block sums of r . s
__global__ __launch_bounds__(kBlock) void k_adi_vupdate(double* __restrict__ v, const double* __restrict__ s2,
                                                       const double* __restrict__ s, double omega, long long N,
                                                       const double* __restrict__ r, double* __restrict__ partial,
                                                       const int* __restrict__ flag) {
  if (flag && *flag) return;
  const long long i = (long long)blockIdx.x * kBlock + threadIdx.x;
  double dot = 0.0;
  if (i < N) {
    v[i] += omega * (s2[i] - s[i]);
    if (partial) dot = r[i] * s[i];
  }
  if (partial) {
    const double sum = block_sum(dot);
    if (threadIdx.x == 0) partial[blockIdx.x] = sum;
  }
}

// Band of a dense symmetric n x n matrix: [n][even_up(2p+1)], entry (i, i+k-p).
std::vector<double> band_of(const std::vector<double>& X, int n, int p) {
  const int W = 2 * p + 1, WP = even_up(W);
  std::vector<double> b((size_t)n * WP, 0.0);
  for (int i = 0; i < n; ++i)
    for (int k = 0; k < W; ++k) {
      const int j = i + k - p;
      if (j >= 0 && j < n) b[(size_t)i * WP + k] = X[(size_t)i * n + j];
    }
  return b;
}

// Lower band Cholesky of cK K + w M (bands as of band_of): [n][p+1], entry (i, i-k),
// the diagonal stored as its reciprocal.
bool band_cholesky(const std::vector<double>& K, const std::vector<double>& M, double cK, double w, int n, int p,
                   double* L) {
  const int W = even_up(2 * p + 1), WL = p + 1;
  auto a = [&](int i, int j) -> double {  // entry (i, j), |i - j| <= p
    const int k = j - i + p;
    return cK * K[(size_t)i * W + k] + w * M[(size_t)i * W + k];
  };
  auto l = [&](int i, int j) -> double& { return L[(size_t)i * WL + (i - j)]; };
  for (int j = 0; j < n; ++j) {
    double s = a(j, j);
    for (int k = std::max(0, j - p); k < j; ++k) s -= l(j, k) * l(j, k);
    if (!(s > 0.0)) return false;
    const double ljj = std::sqrt(s);
    l(j, j) = ljj;
    for (int i = j + 1; i <= std::min(n - 1, j + p); ++i) {
      double v = a(i, j);
      for (int k = std::max(0, i - p); k < j; ++k) v -= l(i, k) * l(j, k);
      l(i, j) = v / ljj;
    }
  }
  for (int j = 0; j < n; ++j) l(j, j) = 1.0 / l(j, j);  // the solves multiply by the reciprocal
  return true;
}

// ||T_J|| for the parameters w: the largest |prod_j g_j| over all triples of
// eigenvalues (host threads over the direction-3 eigenvalues).
double error_norm(const std::vector<double>& w, const std::vector<double>& l1, const std::vector<double>& l2,
                  const std::vector<double>& l3) {
  const unsigned hw = std::thread::hardware_concurrency();
  const int T = (int)std::max(1u, std::min(16u, hw));
  std::vector<double> part(T, 0.0);
  std::vector<std::thread> th;
  for (int t = 0; t < T; ++t)
    th.emplace_back([&, t]() {
      double m = 0.0;
      for (size_t c = t; c < l3.size(); c += T)
        for (double b2 : l2)
          for (double a1 : l1) {
            const double s = a1 + b2 + l3[c];
            double g = 1.0;
            for (double om : w) g *= 1.0 - 2.0 * om * om * s / ((om + a1) * (om + b2) * (om + l3[c]));
            m = std::max(m, std::fabs(g));
          }
      part[t] = m;
    });
  for (auto& x : th) x.join();
  return *std::max_element(part.begin(), part.end());
}

template <int P, int DIR>
igafd_status band_apply(igafd_ctx* c, const double* Bd, double ca, const double* x, const double* x2, double c2,
                        const double* z, double cz, double* y, const int* flag) {
  hipLaunchKernelGGL((k_band_apply<P, DIR>), dim3((unsigned)((c->N + kBlock - 1) / kBlock)), dim3(kBlock), 0, c->stream,
                     Bd, ca, x, x2, c2, z, cz, y, c->n[0], c->n[1], c->n[2], flag);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

template <int P, int DIR>
igafd_status line_solve(igafd_ctx* c, const double* L, double alpha, const double* x, double* y, const int* flag) {
  const long long lines = DIR == 0 ? (long long)c->n[1] * c->n[2] : DIR == 1 ? (long long)c->n[0] * c->n[2]
                                                                            : (long long)c->n[0] * c->n[1];
  const int len = c->n[DIR];
  const dim3 grid((unsigned)((lines + kLineBlock - 1) / kLineBlock));
  const size_t lds = sizeof(double) * (size_t)len * (P + 1);
  if (lds > 64 * 1024) {
    set_error("ADI line too long for the LDS-staged factor");
    return IGAFD_ERR_ARG;
  }
  hipLaunchKernelGGL((k_line_solve<P, DIR>), grid, dim3(kLineBlock), lds, c->stream, L, alpha, x, y, c->n[0], c->n[1],
                     c->n[2], len, flag);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

long long adi_lines(const igafd_ctx* c, int dir) { return c->N / c->n[dir]; }

// Lines per block of a fused sub-step: 32, or 16 where 32 do not fit in LDS or
// would not all be resident at once (a second round of blocks doubles a
// latency-bound launch; 16 lines read 128-byte runs); 0: not even 16 fit.
template <int P>
int lines_per_block(const igafd_ctx* c, int dir, int mode) {
  for (int lt : {32, 16}) {
    const size_t lds = adi_lds<P>(mode, lt, c->n[dir]);
    if (lds > kAdiLds) continue;
    if (lt == 16 || (adi_lines(c, dir) + lt - 1) / lt <= device_cus() * (long long)(kAdiLds / lds)) return lt;
  }
  return 0;
}

// Dynamic LDS above 64 KB needs the kernel attribute; set at setup (never inside a
// launch sequence that may be captured) for the sub-steps of this problem that use
// more, to the largest size that any problem's launch uses.
template <int P, int DIR, int MODE>
igafd_status lds_attr1(const igafd_ctx* c) {
  const int lt = lines_per_block<P>(c, DIR, MODE);
  if (lt == 0 || adi_lds<P>(MODE, lt, c->n[DIR]) <= 64 * 1024) return IGAFD_OK;
  for (const void* fn : {(const void*)&k_adi<P, DIR, 32, MODE>, (const void*)&k_adi<P, DIR, 16, MODE>})
    IGAFD_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAdiLds));
  return IGAFD_OK;
}

template <int P>
igafd_status lds_attr(const igafd_ctx* c) {
  igafd_status s;
  if ((s = lds_attr1<P, 1, ADI_INIT>(c)) != IGAFD_OK || (s = lds_attr1<P, 2, ADI_INIT>(c)) != IGAFD_OK ||
      (s = lds_attr1<P, 1, ADI_A>(c)) != IGAFD_OK || (s = lds_attr1<P, 0, ADI_B>(c)) != IGAFD_OK ||
      (s = lds_attr1<P, 1, ADI_C>(c)) != IGAFD_OK || (s = lds_attr1<P, 2, ADI_D>(c)) != IGAFD_OK)
    return s;
  return IGAFD_OK;
}

// one fused sub-step; slot: 0 = M_d, j + 1 = K_d + omega_j M_d
template <int P, int DIR, int MODE>
igafd_status sub_step(igafd_ctx* c, AdiArgs g, int slot, const int* flag) {
  const int lt = lines_per_block<P>(c, DIR, MODE), len = c->n[DIR];
  const double* fac = c->adi->rows[DIR] + (size_t)slot * 2 * adi_rows(len) * even_up(P + 1);
  g.n1 = c->n[0];
  g.n2 = c->n[1];
  g.n3 = c->n[2];
  g.flag = flag;
  const dim3 grid((unsigned)((adi_lines(c, DIR) + lt - 1) / lt));
  const size_t lds = adi_lds<P>(MODE, lt, len);
  if (lt == 32)
    hipLaunchKernelGGL((k_adi<P, DIR, 32, MODE>), grid, dim3(kAdiThreads), lds, c->stream, g, fac);
  else
    hipLaunchKernelGGL((k_adi<P, DIR, 16, MODE>), grid, dim3(kAdiThreads), lds, c->stream, g, fac);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status adi_lds_attr(const igafd_ctx* c) {
  switch (c->p) {
#define IGAFD_P(P) \
  case P:          \
    return lds_attr<P>(c);
    IGAFD_P(1) IGAFD_P(2) IGAFD_P(3) IGAFD_P(4) IGAFD_P(5) IGAFD_P(6)
#undef IGAFD_P
    default:
      set_error("unsupported degree");
      return IGAFD_ERR_ARG;
  }
}

// blocks of the fused last sub-step; 0: it runs unfused (lines too long, or more
// blocks than the partial-sum buffer holds)
template <int P>
int dot_blocks_p(const igafd_ctx* c) {
  const int lt = lines_per_block<P>(c, 2, ADI_D);
  const long long blocks = lt ? (adi_lines(c, 2) + lt - 1) / lt : 0;
  return lt && blocks <= c->npartial ? (int)blocks : 0;
}

int vblocks_of(const igafd_ctx* c) { return (int)((c->N + kBlock - 1) / kBlock); }

// s = P_J^-1 r by the steps of Alg. "3D ADI method" (s_0 = v_0 = 0)
template <int P>
igafd_status apply_p(igafd_ctx* c, const double* r, double* s, double* partial, const int* flag) {
  igafd_adi* a = c->adi;
  const long long N = c->N;
  double* rt = a->work;
  double* v = rt + N;
  double* u = v + N;
  double* t1 = u + N;
  double* t2 = t1 + N;
  const int n1 = c->n[0], n2 = c->n[1], n3 = c->n[2];
  auto facM = [&](int d) { return a->fac[d]; };
  auto facW = [&](int d, int j) { return a->fac[d] + (size_t)(j + 1) * (d == 0 ? n1 : d == 1 ? n2 : n3) * (P + 1); };
  igafd_status st;
#define IGAFD_T(x)               \
  if ((st = (x)) != IGAFD_OK) \
    return st;
  const bool fa = lines_per_block<P>(c, 1, ADI_A) > 0, fb = lines_per_block<P>(c, 0, ADI_B) > 0;
  const bool fc = lines_per_block<P>(c, 1, ADI_C) > 0, fd = dot_blocks_p<P>(c) > 0;
  const bool all = fa && fb && fc && fd;  // no sub-step reads the zeros of the first step
  // r~ = 2 (I x M2 x M3)^-1 r
  if (lines_per_block<P>(c, 1, ADI_INIT) > 0) {
    AdiArgs g{};
    g.x0 = r;
    g.c = 2.0;
    g.y0 = t1;
    IGAFD_T((sub_step<P, 1, ADI_INIT>(c, g, 0, flag)));
  } else {
    IGAFD_T((line_solve<P, 1>(c, facM(1), 2.0, r, t1, flag)));
  }
  if (lines_per_block<P>(c, 2, ADI_INIT) > 0) {
    AdiArgs g{};
    g.x0 = t1;
    g.c = 1.0;
    g.y0 = rt;
    IGAFD_T((sub_step<P, 2, ADI_INIT>(c, g, 0, flag)));
  } else {
    IGAFD_T((line_solve<P, 2>(c, facM(2), 1.0, t1, rt, flag)));
  }
  const unsigned vb = (unsigned)vblocks_of(c);
  if (!all) {
    hipLaunchKernelGGL(k_adi_fill0, dim3(vb), dim3(kBlock), 0, c->stream, s, v, N, flag);
    IGAFD_HIP_CHECK(hipGetLastError());
  }
  const int J = (int)a->omega.size();
  for (int j = 0; j < J; ++j) {
    const double w = a->omega[j];
    const int first = all && j == 0;
    double* dots = j + 1 == J ? partial : nullptr;
    // u_j = (I x M2^-1 K2 x I) s_{j-1}
    if (first) {  // zero
    } else if (fa) {
      AdiArgs g{};
      g.x0 = s;
      g.band0 = a->bandK[1];
      g.y0 = u;
      IGAFD_T((sub_step<P, 1, ADI_A>(c, g, 0, flag)));
    } else {
      IGAFD_T((band_apply<P, 1>(c, a->bandK[1], 1.0, s, nullptr, 0.0, nullptr, 0.0, t1, flag)));
      IGAFD_T((line_solve<P, 1>(c, facM(1), 1.0, t1, u, flag)));
    }
    // r*_j = r~ - ((K1 - w M1) x I x I) s_{j-1} - (2 M1 x I x I)(u_j + v_j); s*_j
    const double* kw1 = a->bandKw1 + (size_t)j * n1 * even_up(2 * P + 1);
    if (fb) {
      AdiArgs g{};
      g.x0 = s;
      g.x1 = u;
      g.x2 = v;
      g.x3 = rt;
      g.band0 = kw1;
      g.band1 = a->bandM[0];
      g.y0 = t1;
      g.first = first;
      IGAFD_T((sub_step<P, 0, ADI_B>(c, g, j + 1, flag)));
    } else {
      IGAFD_T((band_apply<P, 0>(c, kw1, -1.0, s, nullptr, 0.0, rt, 1.0, t1, flag)));
      IGAFD_T((band_apply<P, 0>(c, a->bandM[0], -2.0, u, v, 1.0, t1, 1.0, t1, flag)));
      IGAFD_T((line_solve<P, 0>(c, facW(0, j), 1.0, t1, t1, flag)));
    }
    // r**_j = (I x M2 x I)(u_j + w s*_j); s**_j
    if (fc) {
      AdiArgs g{};
      g.x0 = u;
      g.x1 = t1;
      g.c = w;
      g.band0 = a->bandM[1];
      g.y0 = t2;
      g.first = first;
      IGAFD_T((sub_step<P, 1, ADI_C>(c, g, j + 1, flag)));
    } else {
      IGAFD_T((band_apply<P, 1>(c, a->bandM[1], 1.0, u, t1, w, nullptr, 0.0, t2, flag)));
      IGAFD_T((line_solve<P, 1>(c, facW(1, j), 1.0, t2, t2, flag)));
    }
    // b_j = v_j + w s**_j; r_j = (I x I x M3) b_j; s_j; v_{j+1} = b_j - w s_j
    if (fd) {
      AdiArgs g{};
      g.x0 = v;
      g.x1 = t2;
      g.x2 = r;
      g.c = w;
      g.band0 = a->bandM[2];
      g.y0 = s;
      g.y1 = v;
      g.first = first;
      g.partial = dots;
      IGAFD_T((sub_step<P, 2, ADI_D>(c, g, j + 1, flag)));
    } else {
      IGAFD_T((band_apply<P, 2>(c, a->bandM[2], 1.0, v, t2, w, nullptr, 0.0, t1, flag)));
      IGAFD_T((line_solve<P, 2>(c, facW(2, j), 1.0, t1, s, flag)));
      hipLaunchKernelGGL(k_adi_vupdate, dim3(vb), dim3(kBlock), 0, c->stream, v, t2, s, w, N, r, dots, flag);
      IGAFD_HIP_CHECK(hipGetLastError());
    }
  }
#undef IGAFD_T
  if (J == 0 && partial) {
    set_error("internal: ADI without steps");
    return IGAFD_ERR_ARG;
  }
  (void)n3;
  return IGAFD_OK;
}

}  // namespace

// block sums of (r, s) that adi_apply writes
int adi_dot_blocks(const igafd_ctx* c) {
  int b = 0;
  switch (c->p) {
#define IGAFD_P(P)           \
  case P:                    \
    b = dot_blocks_p<P>(c);  \
    break;
    IGAFD_P(1) IGAFD_P(2) IGAFD_P(3) IGAFD_P(4) IGAFD_P(5) IGAFD_P(6)
#undef IGAFD_P
    default:
      break;
  }
  return b ? b : (int)((c->N + kBlock - 1) / kBlock);
}

void adi_free(igafd_ctx* c) {
  igafd_adi* a = c->adi;
  if (!a) return;
  if (a->tables) (void)hipFree(a->tables);
  if (a->work) (void)hipFree(a->work);
  delete a;
  c->adi = nullptr;
}

// eq. greedy2: the omega >= 0 minimising |g(omega; l1, l2, l3)|.  g = 0 at the
// positive roots of f(w) = w^3 - S w^2 + e2 w + e3 (none or two); the smaller
// one is taken.  f(0) = e3 > 0 and f has its local minimum at
// w+ = (S + sqrt(S^2 - 3 e2)) / 3: roots exist iff f(w+) <= 0, and the smaller
// lies between max(0, w-) (the local maximum) and w+.  Without roots g > 0 and
// its minimum is at the one positive root of w^3 - e2 w - 2 e3 (where
// 2 S w^2 / prod(w + l_d) peaks).  Both by bisection to the last bit.
double best_parameter(double l1, double l2, double l3) {
  const double S = l1 + l2 + l3, e2 = l1 * l2 + l1 * l3 + l2 * l3, e3 = l1 * l2 * l3;
  auto bisect = [](auto f, double lo, double hi) {  // f(lo) > 0 >= f(hi) or f(lo) < 0 <= f(hi)
    const bool up = f(lo) < 0.0;
    for (int it = 0; it < 200; ++it) {
      const double mid = 0.5 * (lo + hi);
      if (mid <= lo || mid >= hi) break;
      if ((f(mid) < 0.0) == up)
        lo = mid;
      else
        hi = mid;
    }
    return 0.5 * (lo + hi);
  };
  auto f = [&](double w) { return ((w - S) * w + e2) * w + e3; };
  const double disc = std::sqrt(std::max(0.0, S * S - 3.0 * e2));
  const double wp = (S + disc) / 3.0, wm = std::max(0.0, (S - disc) / 3.0);
  if (f(wp) <= 0.0) return bisect(f, wm, wp);
  auto q = [&](double w) { return (w * w - e2) * w - 2.0 * e3; };
  double hi = std::sqrt(e2) + std::cbrt(2.0 * e3) + 1e-300;
  while (q(hi) <= 0.0) hi *= 2.0;
  return bisect(q, 0.0, hi);
}

// Greedy parameters (eq. greedy1/2): after k steps, the triple of largest
// |prod_j g_j| over the eigenvalue triples (the first in (k3, k2, k1) order on
// ties) picks omega_{k+1} = best_parameter(triple); the first parameter is
// sqrt(a b).  Stops once max |prod g_j| <= eps or at J0 steps.  The products
// are kept per triple (n1 n2 n3 doubles on the host, threads over k3).
igafd_status greedy_parameters(const igafd_ctx* c, double a, double b, double eps, int J0, std::vector<double>* w,
                               double* rho) {
  const std::vector<double>&l1 = c->dir[0].lam, &l2 = c->dir[1].lam, &l3 = c->dir[2].lam;
  const size_t n1 = l1.size(), n2 = l2.size(), n3 = l3.size(), total = n1 * n2 * n3;
  if (total > (size_t(1) << 28)) {
    set_error("greedy ADI parameters: too many eigenvalue triples (more than 2^28)");
    return IGAFD_ERR_ARG;
  }
  std::vector<double> G(total, 1.0);
  const unsigned hw = std::thread::hardware_concurrency();
  const int T = (int)std::max(1u, std::min(16u, hw));
  w->assign(1, std::sqrt(a * b));
  for (;;) {
    const double om = w->back();
    std::vector<double> best(T, -1.0);
    std::vector<size_t> at(T, 0);
    std::vector<std::thread> th;
    for (int t = 0; t < T; ++t)
      th.emplace_back([&, t]() {
        for (size_t k3 = t; k3 < n3; k3 += T)
          for (size_t k2 = 0; k2 < n2; ++k2)
            for (size_t k1 = 0; k1 < n1; ++k1) {
              const size_t i = (k3 * n2 + k2) * n1 + k1;
              const double s = l1[k1] + l2[k2] + l3[k3];
              G[i] = G[i] * (1.0 - 2.0 * om * om * s / ((om + l1[k1]) * (om + l2[k2]) * (om + l3[k3])));
              const double v = std::fabs(G[i]);
              if (v > best[t] || (v == best[t] && i < at[t])) {
                best[t] = v;
                at[t] = i;
              }
            }
      });
    for (auto& x : th) x.join();
    int tb = 0;
    for (int t = 1; t < T; ++t)
      if (best[t] > best[tb] || (best[t] == best[tb] && at[t] < at[tb])) tb = t;
    *rho = best[tb];
    if (*rho <= eps || (int)w->size() >= J0) return IGAFD_OK;
    const size_t i = at[tb];
    const size_t k1 = i % n1, k2 = (i / n1) % n2, k3 = i / (n1 * n2);
    w->push_back(best_parameter(l1[k1], l2[k2], l3[k3]));
  }
}

igafd_status adi_setup(igafd_ctx* c, double eps, int rule) {
  if (c->dim != 3) {
    set_error("the three-variable ADI is for 3D problems");
    return IGAFD_ERR_ARG;
  }
  if (!(eps > 0.0 && eps < 1.0)) {
    set_error("ADI tolerance must lie in (0, 1)");
    return IGAFD_ERR_ARG;
  }
  for (int d = 0; d < 3; ++d)
    if (c->dir[d].lam.empty()) {
      set_error("this context holds no univariate eigenvalues");
      return IGAFD_ERR_ARG;
    }
  const int p = c->p;
  double a = c->dir[0].lam.front(), b = c->dir[0].lam.back();
  for (int d = 0; d < 3; ++d) {
    a = std::min(a, *std::min_element(c->dir[d].lam.begin(), c->dir[d].lam.end()));
    b = std::max(b, *std::max_element(c->dir[d].lam.begin(), c->dir[d].lam.end()));
  }
  const int J0 = std::max(1, (int)std::ceil(1.16 * std::log(b / a) * std::log(1.0 / eps)));
  std::vector<double> w;
  double rho = 1.0;
  if (rule == kAdiGreedy) {
    const igafd_status gs = greedy_parameters(c, a, b, eps, J0, &w, &rho);
    if (gs != IGAFD_OK) return gs;
  } else {
    for (int J = 1; J <= J0; ++J) {
      w.assign(J, 0.0);
      for (int j = 0; j < J; ++j) w[j] = J == 1 ? std::sqrt(a * b) : a * std::pow(b / a, (double)j / (J - 1));
      rho = error_norm(w, c->dir[0].lam, c->dir[1].lam, c->dir[2].lam);
      if (rho <= eps) break;
    }
  }
  std::unique_ptr<igafd_adi> st(new igafd_adi());
  st->eps = eps;
  st->rho = rho;
  st->omega = w;
  st->J0 = J0;
  const int W = even_up(2 * p + 1), WL = p + 1, J = (int)w.size();
  // device buffers are owned by st until it is installed: free them on failure
  struct Guard {
    igafd_adi* a;
    ~Guard() {
      if (!a) return;
      if (a->tables) (void)hipFree(a->tables);
      if (a->work) (void)hipFree(a->work);
    }
  } guard{st.get()};
  // every table in one host array, each 256-byte aligned, for one allocation and one copy
  std::vector<double> host;
  std::vector<std::pair<const double**, size_t>> parts;  // the pointer of a table, its place
  auto add = [&](const double** p, size_t count) {
    parts.push_back({p, host.size()});
    host.resize((host.size() + count + 31) / 32 * 32);
    return host.data() + parts.back().second;  // until the next table is added
  };
  for (int d = 0; d < 3; ++d) {
    const int n = c->dir[d].n;
    const std::vector<double> bK = band_of(c->dir[d].K, n, p), bM = band_of(c->dir[d].M, n, p);
    std::copy(bK.begin(), bK.end(), add(&st->bandK[d], bK.size()));
    std::copy(bM.begin(), bM.end(), add(&st->bandM[d], bM.size()));
    const size_t slot = (size_t)n * WL;
    double* fac = add(&st->fac[d], (J + 1) * slot);
    bool ok = band_cholesky(bK, bM, 0.0, 1.0, n, p, fac);
    for (int j = 0; j < J && ok; ++j) ok = band_cholesky(bK, bM, 1.0, w[j], n, p, fac + (j + 1) * slot);
    if (!ok) {
      set_error("band Cholesky of K_d + omega M_d failed");
      return IGAFD_ERR_NOT_SPD;
    }
    // the sweeps' rows (adi_sweep): forward 1/L_ii, L_{i+k,i}/L_{i+k,i+k}; backward, i from
    // the end after the zero rows, 1/L_ii, L_{i,i-k}/L_{i-k,i-k}
    const int RP = even_up(WL), R = adi_rows(n);
    double* rows = add(&st->rows[d], (size_t)(J + 1) * 2 * R * RP);
    fac = host.data() + parts[parts.size() - 2].second;
    for (int j = 0; j <= J; ++j)
      for (int i = 0; i < n; ++i) {
        const double* f = fac + j * slot;
        double* fw = rows + ((size_t)j * 2 * R + i) * RP;
        double* bw = rows + ((size_t)j * 2 * R + R + (R - 1 - i)) * RP;
        fw[0] = bw[0] = f[(size_t)i * WL];
        for (int k = 1; k <= p; ++k) {
          if (i + k < n) fw[k] = f[(size_t)(i + k) * WL + k] * f[(size_t)(i + k) * WL];
          if (i - k >= 0) bw[k] = f[(size_t)i * WL + k] * f[(size_t)(i - k) * WL];
        }
      }
    if (d > 0) continue;
    double* kw = add(&st->bandKw1, (size_t)J * n * W);  // K1 - omega_j M1 per parameter
    for (int j = 0; j < J; ++j)
      for (size_t e = 0; e < bK.size(); ++e) kw[(size_t)j * n * W + e] = bK[e] - w[j] * bM[e];
  }
  IGAFD_HIP_CHECK(device_malloc((void**)&st->tables, sizeof(double) * host.size()));
  IGAFD_HIP_CHECK(hipMemcpy(st->tables, host.data(), sizeof(double) * host.size(), hipMemcpyHostToDevice));
  for (const auto& part : parts) *part.first = st->tables + part.second;
  IGAFD_HIP_CHECK(device_malloc((void**)&st->work, sizeof(double) * 5 * (size_t)c->N));
  igafd_status sa = adi_lds_attr(c);
  if (sa != IGAFD_OK) return sa;
  adi_free(c);
  guard.a = nullptr;
  c->adi = st.release();
  return IGAFD_OK;
}

igafd_status adi_apply(igafd_ctx* c, int prec, const double* r, double* s, const double* S, double* partial,
                       const int* flag) {
  if (prec != IGAFD_FP64) {
    set_error("the ADI preconditioner runs in FP64 only");
    return IGAFD_ERR_ARG;
  }
  if (S) {
    set_error("the scaled preconditioner is not defined with ADI");
    return IGAFD_ERR_ARG;
  }
  if (partial && adi_dot_blocks(c) > c->npartial) {
    set_error("internal: ADI grid larger than the partial-sum buffer");
    return IGAFD_ERR_ARG;
  }
  switch (c->p) {
#define IGAFD_P(P) \
  case P:          \
    return apply_p<P>(c, r, s, partial, flag);
    IGAFD_P(1) IGAFD_P(2) IGAFD_P(3) IGAFD_P(4) IGAFD_P(5) IGAFD_P(6)
#undef IGAFD_P
    default:
      set_error("unsupported degree");
      return IGAFD_ERR_ARG;
  }
}

}  // namespace igafd
