// Device assembly of the Galerkin stiffness matrix A and of the load vector b.
//
// Paper Sec. 2.1 eq. A / eq. Q: A_ij = int_[0,1]^d grad(B_i)^T Q grad(B_j) with
// Q = |det J| J^-1 K J^-T (J_ij = dF_i/dxi_j), by the tensor (p+1)-point Gauss
// rule on every element.  Only the upper half of the stencil is stored: plane h
// holds offset center + h of the (2p+1)^d stencil, indexed by the row.
//
// Element by element (k_assemble, k_load): one workgroup per element, local
// matrix by sum factorisation, added into the band in (p+1)^d colour classes.
//
// Across the elements (3D contexts that keep the learned-scaling features):
// the Gauss sums are taken one direction at a time over the whole domain.
//   1. k_contract3: a thread owns one column of Gauss points (q1, q2), walks
//      q3, evaluates C = w Q (Q = kappa adj(J) adj(J)^T / |det J|, no inverse)
//      and contracts it with the pairs of direction-3 functions,
//   2. k_contract12: a block owns one direction-3 pair and a run of
//      direction-1 functions; it walks q2, contracts the direction-2 pairs and
//      then, per finished pair of grid lines, direction 1, and stores the band.
// The contraction of a direction walks the functions in order: an element adds
// to the pairs of its p+1 functions, held in registers, and the pairs of the
// first of them are complete when the walk leaves it.  Every entry is written
// by one thread, once.  Features and load vectors go the same way.
// Measured, warped cube with kappa: 112^3, p = 4: 15.1 ms for the band (4.3 GB)
// against 197 ms by colours (which read, add to and write it); load vector 2.9
// against 22.6 ms; 16^3, p = 3: 0.21 ms in 10 launches against 1.7 ms in 64.
//
// Both sums are in a fixed order (bitwise reproducible, no atomics), but not in
// the same one: the entries differ in their last bits.  A context's order is a
// matter of its features alone, whatever precision its solves use: contexts
// without them keep the element order, so that their results stay what they
// were bit for bit (flexible CG with plain BF16 applies turns a last bit of A or
// b into up to 3e-9 of the solution, the iterates taking another path within
// the same tolerance; the other precisions follow to rounding).
#include <algorithm>

#include "internal.h"

namespace igafd {
namespace {

// right-hand side f of igafd_load_vector: kind, amplitude, SINPROD frequencies
struct RhsDesc {
  int kind;
  double amp;
  double k[3];
};

struct Tables {
  const int* first[3];
  const double* qx[3];
  const double* qw[3];
  const double* val[3];
  const double* der[3];
  int n[3];
};

// The arguments of up to 216 launches in a row, which take as long as the host needs
// for them: three pointers more made load vectors of 8^3 to 24^3 elements 4 %
// slower (16^3, p = 3: 327 -> 339 us), so what only others need is not in here.
static_assert(sizeof(Tables) == 15 * sizeof(void*) + 4 * sizeof(int), "argument of the element kernels");

// for the kernels across the elements
struct AcrossTables : Tables {
  const int* at[3];  // at[l][f]: element whose first function is f, or -1 (f < n_l + 2)
};

template <int D>
__device__ inline void map_eval(const GeomDesc& g, const double xi[3], double x[3], double J[3][3]) {
  for (int a = 0; a < 3; ++a) {
    x[a] = xi[a];
    for (int b = 0; b < 3; ++b) J[a][b] = (a == b) ? 1.0 : 0.0;
  }
  if (g.kind == IGAFD_GEOM_RING) {
    const double r = 1.0 + xi[0];
    const double th = 0.5 * M_PI * xi[1];
    double s, c;
    sincos(th, &s, &c);
    x[0] = r * c;
    x[1] = r * s;
    J[0][0] = c;
    J[0][1] = -0.5 * M_PI * r * s;
    J[1][0] = s;
    J[1][1] = 0.5 * M_PI * r * c;
  } else if (g.kind == IGAFD_GEOM_WARPED) {
    for (int k = 0; k < g.nmodes; ++k) {
      double sn[3], dc[3];
      for (int l = 0; l < D; ++l) {
        double s, c;
        sincos(M_PI * g.m[k][l] * xi[l], &s, &c);
        sn[l] = s;
        dc[l] = M_PI * g.m[k][l] * c;
      }
      double prod = 1.0;
      for (int l = 0; l < D; ++l) prod *= sn[l];
      for (int a = 0; a < D; ++a) x[a] += g.amp * g.c[k][a] * prod;
      for (int j = 0; j < D; ++j) {
        double others = dc[j];
        for (int l = 0; l < D; ++l)
          if (l != j) others *= sn[l];
        for (int a = 0; a < D; ++a) J[a][j] += g.amp * g.c[k][a] * others;
      }
    }
  }
}

__device__ inline double kappa_eval(const GeomDesc& g, const double x[3]) {
  if (g.coef_kind == IGAFD_COEF_SINCOS)
    return 1.0 + g.camp * sin(2.0 * M_PI * g.f1 * x[0] + g.phi1) * cos(2.0 * M_PI * g.f2 * x[1] + g.phi2);
  return 1.0;
}

// det J and the cofactor matrix adj(J) (so that J^-1 = adj / det).
template <int D>
__device__ inline double adjugate(const double J[3][3], double A[3][3]) {
  if (D == 2) {
    A[0][0] = J[1][1];
    A[0][1] = -J[0][1];
    A[1][0] = -J[1][0];
    A[1][1] = J[0][0];
    return J[0][0] * J[1][1] - J[0][1] * J[1][0];
  }
  A[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
  A[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
  A[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
  A[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
  A[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
  A[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
  A[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  A[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
  A[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
  return J[0][0] * A[0][0] + J[0][1] * A[1][0] + J[0][2] * A[2][0];
}

template <int D>
__host__ __device__ constexpr int sym_index(int a, int b) {
  return (a == b) ? a : (D == 2 ? 2 : (a + b == 1 ? 3 : (a + b == 2 ? 4 : 5)));
}

// Per-dof statistics of the learned scaling, one element's share: for the
// kChan channels and every local function a = (a1, a2, a3) of
// the element, sum_t B_a(t) v(ch, t) over the element's Gauss points t, where
// v(ch, t) = w_t G_ch(t) (ch < 6: the entries 11, 22, 33, 12, 13, 23 of
// G = |det J| J^-1 J^-T), w_t kappa(t) (ch = 6) or w_t (ch = 7), given in
// vals[ch][t].  The sum is taken one direction at a time (sum
// factorisation: t1, then t2, then t3) and added into acc[8 row + ch] for the
// functions that are dofs; the element's colour class guarantees no other
// block adds to those rows.  F1 (kChan L Q Q3 doubles) and F2 (kChan L L Q3) are
// LDS scratch; vals may share F2's storage (it is last read before F2 is
// written).
constexpr int kChan = 8;
template <int D, int P>
__device__ void feature_sums(const double* vals, const double (*sV)[P + 1][P + 1], const int* first,
                             const Tables& T, double* F1, double* F2, double* __restrict__ acc) {
  constexpr int Q = P + 1, L = P + 1;
  constexpr int Q3 = (D == 3) ? Q : 1;
  constexpr int L3 = (D == 3) ? L : 1;
  constexpr int NQ = Q * Q * Q3;
  const int tid = threadIdx.x;
  for (int idx = tid; idx < kChan * L * Q * Q3; idx += kBlock) {  // F1[c][t2 + Q t3][a1]
    const int c = idx / (L * Q * Q3), r = idx % (L * Q * Q3);
    const int a1 = r % L, t23 = r / L;
    double s = 0.0;
#pragma unroll
    for (int t1 = 0; t1 < Q; ++t1) s += sV[0][t1][a1] * vals[c * NQ + t1 + Q * t23];
    F1[idx] = s;
  }
  __syncthreads();
  for (int idx = tid; idx < kChan * L * L * Q3; idx += kBlock) {  // F2[c][t3][a2][a1]
    const int c = idx / (L * L * Q3), r = idx % (L * L * Q3);
    const int a1 = r % L, a2 = (r / L) % L, t3 = r / (L * L);
    double s = 0.0;
#pragma unroll
    for (int t2 = 0; t2 < Q; ++t2) s += sV[1][t2][a2] * F1[c * (L * Q * Q3) + (t2 + Q * t3) * L + a1];
    F2[idx] = s;
  }
  __syncthreads();
  // one thread per local function: its kChan channel sums, then one
  // read-modify-write of the kChan consecutive doubles of its row (a 64-byte run,
  // instead of kChan scattered 8-byte accesses from as many waves)
  typedef double dpair __attribute__((ext_vector_type(2)));
  constexpr int DOFS = L * L * L3, PER = (DOFS + kBlock - 1) / kBlock;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int r = tid + k * kBlock;
    if (r >= DOFS) break;
    const int a1 = r % L, a2 = (r / L) % L, a3 = r / (L * L);
    const int r1 = first[0] + a1 - 1, r2 = first[1] + a2 - 1, r3 = (D == 3) ? first[2] + a3 - 1 : 0;
    if (r1 < 0 || r1 >= T.n[0] || r2 < 0 || r2 >= T.n[1] || r3 < 0 || r3 >= T.n[2]) continue;
    dpair* row = reinterpret_cast<dpair*>(acc + 8 * (r1 + (long long)T.n[0] * (r2 + (long long)T.n[1] * r3)));
    // four channels at a time (fewer registers than eight sums and their old values)
#pragma unroll
    for (int h = 0; h < kChan; h += 4) {
      const dpair o0 = row[h / 2], o1 = row[h / 2 + 1];
      double sv[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        double s = 0.0;
#pragma unroll
        for (int t3 = 0; t3 < Q3; ++t3) s += sV[2][t3][a3] * F2[(h + c) * (L * L * Q3) + (t3 * L + a2) * L + a1];
        sv[c] = s;
      }
      row[h / 2] = dpair{o0.x + sv[0], o0.y + sv[1]};
      row[h / 2 + 1] = dpair{o1.x + sv[2], o1.y + sv[3]};
    }
  }
  __syncthreads();
}

// FEAT = 1 (2D; 3D contexts with features are assembled across the elements):
// also the per-dof feature sums of the learned scaling into acc (8 doubles per
// dof), from the same Gauss-point evaluation of the map.
template <int D, int P, int FEAT>
__global__ __launch_bounds__(kBlock, (D == 3 && P <= 4) ? 5 : 1) void k_assemble(Tables T, GeomDesc g, double* __restrict__ band,
                                                     long long Ns, int c1, int c2, int c3, int m1, int m2,
                                                     int* __restrict__ err, double* __restrict__ acc) {
  constexpr int Q = P + 1, L = P + 1;
  constexpr int Q3 = (D == 3) ? Q : 1;
  constexpr int L3 = (D == 3) ? L : 1;
  constexpr int NQ = Q * Q * Q3;
  constexpr int NC = (D == 3) ? 6 : 3;
  constexpr int NAB = D * D;
  constexpr int W = 2 * P + 1;
  constexpr int S = (D == 3) ? W * W * W : W * W;
  constexpr int CENTER = (S - 1) / 2;
  constexpr int R3 = (D == 3) ? P : 0;

  __shared__ double sC[NC][NQ];
  __shared__ double sV[3][Q][L];
  __shared__ double sD[3][Q][L];
  __shared__ double sH[NAB][Q * Q];
  __shared__ double sG[NAB][L * L][Q];
  __shared__ int sFirst[3];
  // features: kappa and the weight per point, F2 of the contraction (F1 lives in sG)
  static_assert(!FEAT || D == 2, "features with A by elements in 2D only");
  __shared__ double sKap[FEAT ? NQ : 1], sW[FEAT ? NQ : 1];
  __shared__ double sF2[FEAT ? kChan * L * L * Q3 : 1];  // the channel values, then F2
  static_assert(!FEAT || NAB * L * L * Q >= kChan * L * Q * Q3, "feature scratch F1 must fit in sG");
  static_assert(!FEAT || L * L * Q3 >= NQ, "channel values must fit in sF2");

  int bid = blockIdx.x;
  const int j1 = bid % m1;
  bid /= m1;
  const int j2 = bid % m2;
  const int j3 = bid / m2;
  const int e[3] = {c1 + j1 * (P + 1), c2 + j2 * (P + 1), (D == 3) ? c3 + j3 * (P + 1) : 0};
  const int tid = threadIdx.x;

  for (int idx = tid; idx < 3 * Q * L; idx += kBlock) {
    const int l = idx / (Q * L), t = (idx / L) % Q, a = idx % L;
    if (l < D) {
      sV[l][t][a] = T.val[l][(e[l] * Q + t) * L + a];
      sD[l][t][a] = T.der[l][(e[l] * Q + t) * L + a];
    } else {
      sV[l][t][a] = (t == 0 && a == 0) ? 1.0 : 0.0;
      sD[l][t][a] = 0.0;
    }
  }
  if (tid < 3) sFirst[tid] = (tid < D) ? T.first[tid][e[tid]] : 1;

  for (int t = tid; t < NQ; t += kBlock) {
    const int t1 = t % Q, t2 = (t / Q) % Q, t3 = t / (Q * Q);
    double xi[3] = {T.qx[0][e[0] * Q + t1], T.qx[1][e[1] * Q + t2], 0.0};
    double w = T.qw[0][e[0] * Q + t1] * T.qw[1][e[1] * Q + t2];
    if (D == 3) {
      xi[2] = T.qx[2][e[2] * Q + t3];
      w *= T.qw[2][e[2] * Q + t3];
    }
    double x[3], J[3][3], A[3][3];
    map_eval<D>(g, xi, x, J);
    const double det = adjugate<D>(J, A);
    if (!(det > 0.0)) *err = 1;
    const double kap = kappa_eval(g, x);
    const double f = w * kap / fabs(det);
    for (int a = 0; a < D; ++a)
      for (int b = a; b < D; ++b) {
        double s = 0.0;
        for (int k = 0; k < D; ++k) s += A[a][k] * A[b][k];
        sC[sym_index<D>(a, b)][t] = f * s;
      }
    if (FEAT) {
      sKap[t] = kap;
      sW[t] = w;
    }
  }
  __syncthreads();
  if (FEAT) {
    // the channel values at the Gauss points: w G_ab = C_ab / kappa; the channel
    // order is (11, 22, 33, 12, 13, 23, kappa, 1), those of direction 3 zero
    for (int idx = tid; idx < kChan * NQ; idx += kBlock) {
      const int ch = idx / NQ, t = idx % NQ;
      double v;
      if (ch == 6)
        v = sW[t] * sKap[t];
      else if (ch == 7)
        v = sW[t];
      else if (ch == 2 || ch > 3)
        v = 0.0;
      else
        v = sC[ch == 3 ? sym_index<D>(0, 1) : sym_index<D>(ch, ch)][t] / sKap[t];
      sF2[idx] = v;
    }
    __syncthreads();
    feature_sums<D, P>(sF2, sV, sFirst, T, &sG[0][0][0], sF2, acc);
  }

  for (int a3 = 0; a3 < L3; ++a3) {
    for (int b3 = a3; b3 < L3; ++b3) {
      // H[ab][t1 + Q t2] = sum_t3 C_ab(t) phi3(a3) phi3(b3)
      for (int idx = tid; idx < NAB * Q * Q; idx += kBlock) {
        const int ab = idx / (Q * Q), t12 = idx % (Q * Q);
        const int a = ab / D, b = ab % D;
        const int ci = sym_index<D>(a, b);
        double s = 0.0;
#pragma unroll
        for (int t3 = 0; t3 < Q3; ++t3) {
          const double fa = (a == 2) ? sD[2][t3][a3] : sV[2][t3][a3];
          const double fb = (b == 2) ? sD[2][t3][b3] : sV[2][t3][b3];
          s += sC[ci][t12 + Q * Q * t3] * fa * fb;
        }
        sH[ab][t12] = s;
      }
      __syncthreads();
      // G[ab][a2 + L b2][t1] = sum_t2 H[ab][t1 + Q t2] phi2(a2) phi2(b2)
      for (int idx = tid; idx < NAB * L * L * Q; idx += kBlock) {
        const int ab = idx / (L * L * Q), rem = idx % (L * L * Q);
        const int a2b2 = rem / Q, t1 = rem % Q;
        const int a2 = a2b2 % L, b2 = a2b2 / L;
        const int a = ab / D, b = ab % D;
        double s = 0.0;
#pragma unroll
        for (int t2 = 0; t2 < Q; ++t2) {
          const double fa = (a == 1) ? sD[1][t2][a2] : sV[1][t2][a2];
          const double fb = (b == 1) ? sD[1][t2][b2] : sV[1][t2][b2];
          s += sH[ab][t1 + Q * t2] * fa * fb;
        }
        sG[ab][a2b2][t1] = s;
      }
      __syncthreads();
      // local entry (a1 a2 a3 | b1 b2 b3) = sum_ab sum_t1 G phi1(a1) phi1(b1)
      for (int idx = tid; idx < L * L * L * L; idx += kBlock) {
        const int a1 = idx % L, b1 = (idx / L) % L, a2 = (idx / (L * L)) % L, b2 = idx / (L * L * L);
        const int o1 = b1 - a1, o2 = b2 - a2, o3 = b3 - a3;
        if (o3 == 0 && (o2 < 0 || (o2 == 0 && o1 < 0))) continue;  // lower half: not stored
        const int r1 = sFirst[0] + a1 - 1, r2 = sFirst[1] + a2 - 1, r3 = (D == 3) ? sFirst[2] + a3 - 1 : 0;
        const int q1 = r1 + o1, q2 = r2 + o2, q3 = r3 + o3;
        if (r1 < 0 || r1 >= T.n[0] || r2 < 0 || r2 >= T.n[1] || r3 < 0 || r3 >= T.n[2]) continue;
        if (q1 < 0 || q1 >= T.n[0] || q2 < 0 || q2 >= T.n[1] || q3 < 0 || q3 >= T.n[2]) continue;
        double s = 0.0;
#pragma unroll
        for (int ab = 0; ab < NAB; ++ab) {
          const int a = ab / D, b = ab % D;
#pragma unroll
          for (int t1 = 0; t1 < Q; ++t1) {
            const double fa = (a == 0) ? sD[0][t1][a1] : sV[0][t1][a1];
            const double fb = (b == 0) ? sD[0][t1][b1] : sV[0][t1][b1];
            s += sG[ab][a2 + L * b2][t1] * fa * fb;
          }
        }
        const int oidx = ((o3 + R3) * W + (o2 + P)) * W + (o1 + P);
        const long long row = r1 + (long long)T.n[0] * (r2 + (long long)T.n[1] * r3);
        band[(long long)(oidx - CENTER) * Ns + row] += s;
      }
      __syncthreads();
    }
  }
}

// ---- columns of Gauss points ----
// The map on the column (xi1, xi2) of Gauss points: x = base + xi3 e3 + sum_k
// (a c_k sin(pi m_k3 xi3)) m0_k and the Jacobian alike, with the products
// m0 = s1 s2, m1 = s1' s2, m2 = s1 s2' of each mode k held in LDS for the
// thread's column ([k][3][threads]) and the direction-3 factors
// a c_k s3, a c_k s3' (six per point and mode) in a table.
constexpr int kCol = 128;    // columns per block
constexpr int kModePad = 4;  // the modes are padded (zero amplitude) to chunks of this many

struct Modes {
  const double* d12[2];  // [q][K][2]: sin(pi m xi), pi m cos(pi m xi) of directions 1 and 2
  const double* d3;      // [q][K][6]: a c_x s, a c_y s, a c_z s, a c_x s', a c_y s', a c_z s'
  int K;                 // modes, padded to a multiple of kModePad (0: none)
};

struct Column {
  double x0, x1, j00, j01, j10, j11;
};

__device__ inline Column column_of(const GeomDesc& g, double xi1, double xi2) {
  Column c{xi1, xi2, 1.0, 0.0, 0.0, 1.0};
  if (g.kind == IGAFD_GEOM_RING) {
    const double r = 1.0 + xi1;
    double s, co;
    sincos(0.5 * M_PI * xi2, &s, &co);
    c.x0 = r * co;
    c.x1 = r * s;
    c.j00 = co;
    c.j01 = -0.5 * M_PI * r * s;
    c.j10 = s;
    c.j11 = 0.5 * M_PI * r * co;
  }
  return c;
}

// the thread's mode products into its LDS slots (read back by the same thread)
__device__ inline void column_modes(const Modes& m, int q1, int q2, double* sm, int lane) {
  for (int k = 0; k < m.K; ++k) {
    const double* a = m.d12[0] + 2 * ((long long)q1 * m.K + k);
    const double* b = m.d12[1] + 2 * ((long long)q2 * m.K + k);
    double* o = sm + (size_t)(3 * k) * kCol + lane;
    o[0] = a[0] * b[0];
    o[kCol] = a[1] * b[0];
    o[2 * kCol] = a[0] * b[1];
  }
}

// Tables that no kernel below writes, read at wave-uniform indices: the
// constant address space takes them through scalar loads (one value for the
// wave, in scalar registers), also where the compiler cannot prove that the
// kernel's stores leave them alone.
typedef const double __attribute__((address_space(4))) ctab_t;
typedef const int __attribute__((address_space(4))) cidx_t;

// x and J at point q3 of the column
__device__ inline void column_eval(const Column& c, int K, ctab_t* d3, const double* sm, int lane,
                                   int q3, double xi3, double x[3], double J[3][3]) {
  x[0] = c.x0;
  x[1] = c.x1;
  x[2] = xi3;
  J[0][0] = c.j00;
  J[0][1] = c.j01;
  J[0][2] = 0.0;
  J[1][0] = c.j10;
  J[1][1] = c.j11;
  J[1][2] = 0.0;
  J[2][0] = 0.0;
  J[2][1] = 0.0;
  J[2][2] = 1.0;
  ctab_t* t = d3 + 6 * (long long)q3 * K;
  for (int k = 0; k < K; k += kModePad, t += 6 * kModePad) {
    double sv[kModePad][3];
#pragma unroll
    for (int j = 0; j < kModePad; ++j)
#pragma unroll
      for (int i = 0; i < 3; ++i) sv[j][i] = sm[(size_t)(3 * (k + j) + i) * kCol + lane];
#pragma unroll
    for (int j = 0; j < kModePad; ++j)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double c = t[6 * j + a];
        x[a] = fma(c, sv[j][0], x[a]);
        J[a][0] = fma(c, sv[j][1], J[a][0]);
        J[a][1] = fma(c, sv[j][2], J[a][1]);
        J[a][2] = fma(t[6 * j + 3 + a], sv[j][0], J[a][2]);
      }
  }
}

// tables of Modes: one thread per (point, mode) of the three directions
__global__ void k_mode_tables(const double* qx0, const double* qx1, const double* qx2, int nq0, int nq1, int nq2,
                              GeomDesc g, int K, double* d0, double* d1, double* d3) {
  int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  for (int l = 0; l < 3; ++l) {
    const int n = (l == 0 ? nq0 : l == 1 ? nq1 : nq2) * K;
    if (i >= n) {
      i -= n;
      continue;
    }
    const int q = i / K, k = i % K;
    double s = k < g.nmodes ? 1.0 : 0.0, ds = 0.0;
    if (k < g.nmodes) {
      double sn, co;
      sincos(M_PI * g.m[k][l] * (l == 0 ? qx0 : l == 1 ? qx1 : qx2)[q], &sn, &co);
      s = sn;
      ds = M_PI * g.m[k][l] * co;
    }
    if (l < 2) {
      double* o = (l == 0 ? d0 : d1) + 2 * (long long)i;
      o[0] = s;
      o[1] = ds;
    } else {
      for (int a = 0; a < 3; ++a) {
        const double c = k < g.nmodes ? g.amp * g.c[k][a] : 0.0;
        d3[6 * (long long)i + a] = c * s;
        d3[6 * (long long)i + 3 + a] = c * ds;
      }
    }
    return;
  }
}

// The values contracted over the Gauss points: C = w Q (order 11, 12, 22, 33,
// 13, 23), or the feature channels w G (11, 22, 33, 12, 13, 23) and w kappa
// with G = |det J| J^-1 J^-T.  Returns det J.
enum { VAL_C = 0, VAL_FEAT = 1 };
template <int WHAT>
__device__ inline double point_values(const GeomDesc& g, const double x[3], const double J[3][3], double w,
                                      double* v) {
  double A[3][3];
  const double det = adjugate<3>(J, A);
  double s[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) s[a][b] = A[a][0] * A[b][0] + A[a][1] * A[b][1] + A[a][2] * A[b][2];
  const double kap = kappa_eval(g, x);
  if (WHAT == VAL_C) {
    const double f = w * kap / fabs(det);
    v[0] = f * s[0][0];
    v[1] = f * s[0][1];
    v[2] = f * s[1][1];
    v[3] = f * s[2][2];
    v[4] = f * s[0][2];
    v[5] = f * s[1][2];
  } else {
    const double f = w / fabs(det);
    v[0] = f * s[0][0];
    v[1] = f * s[1][1];
    v[2] = f * s[2][2];
    v[3] = f * s[0][1];
    v[4] = f * s[0][2];
    v[5] = f * s[1][2];
    v[6] = w * kap;
  }
  return det;
}

template <int D>
__device__ inline double rhs_eval(const RhsDesc& f, const double x[3]) {
  switch (f.kind) {
    case IGAFD_RHS_SINPROD: {
      double s = f.amp;
      for (int l = 0; l < D; ++l) s *= sin(f.k[l] * M_PI * x[l]);
      return s;
    }
    case IGAFD_RHS_PAPER_POLY: {
      double s = 0.0;
      for (int l = 0; l < D; ++l) s += 2.0 * (x[l] * x[l] - x[l]);
      return f.amp * s;
    }
    case IGAFD_RHS_BUBBLE: {
      double s = 0.0;
      for (int i = 0; i < D; ++i) {
        double pr = 2.0;
        for (int l = 0; l < D; ++l)
          if (l != i) pr *= x[l] * (1.0 - x[l]);
        s += pr;
      }
      return f.amp * s;
    }
    default:
      return f.amp;
  }
}

// Fields of the direction-3 contraction H (per pair (i3, i3 + o), o >= 0, and
// Gauss column): 0..3 = C11 B B, C12 B B, C22 B B, C33 B' B'; 4, 5 = C13 B B',
// C13 B' B; 6, 7 = C23 B B', C23 B' B (first factor: function i3).
constexpr int kFields3 = 8;
constexpr int kFeat = 7;

// Direction-3 contraction.  A block owns kCol columns (q1, q2) and a run of
// `len` functions i3 of [base, end) and walks the elements below them (p more
// than the run is long, so a longer run repeats less of the evaluation).  Its
// two halves hold the same columns: each evaluates the map at every second
// Gauss point of an element and hands the six values over in LDS, and each
// sums four of the eight fields, 2 (p+1)(p+2) accumulators per thread, which
// stay within the register file up to p = 6.
// Bound by the FP64 issue rate of the evaluation (about 430 instructions per
// point with a warped map and kappa, 8 modes) and of the pair sums (85 per point
// and half at p = 4): 112^3, p = 4: 7.6 ms in all, at two waves per SIMD;
// one map evaluation per half and point, each half for
// itself, took 9.6 ms.
template <int P>
__global__ __launch_bounds__(2 * kCol, P <= 5 ? 2 : 1) void k_contract3(
    AcrossTables T, GeomDesc g, Modes md, int nq1, int nq2, cidx_t* at, ctab_t* qx, ctab_t* qw, ctab_t* val,
    ctab_t* der, ctab_t* d3, int base, int end, int len, double* __restrict__ H,
    int* __restrict__ err) {
  extern __shared__ double sm[];
  constexpr int Q = P + 1, NP = (P + 1) * (P + 2) / 2;
  double* sV = sm;                  // [2 buffers][2 points][6][kCol]
  double* sM = sm + 24 * kCol;      // [K][3][kCol]
  const int lane = threadIdx.x % kCol;
  // the half of the C13, C23 fields (the first: C11, C12, C22, C33); wave-uniform
  const int mixed = __builtin_amdgcn_readfirstlane(threadIdx.x / kCol);
  const long long nq12 = (long long)nq1 * nq2;
  const long long q12 = (long long)blockIdx.x * kCol + lane;
  const bool live = q12 < nq12;
  const int c0 = base + (int)blockIdx.y * len, c1 = min(c0 + len, end);
  const int q1 = live ? (int)(q12 % nq1) : 0, q2 = live ? (int)(q12 / nq1) : 0;
  const Column col = column_of(g, T.qx[0][q1], T.qx[1][q2]);
  if (!mixed) column_modes(md, q1, q2, sM, lane);
  const double w12 = T.qw[0][q1] * T.qw[1][q2];
  double acc[4][NP];  // slot of the pair (a, a + o): a (P + 1) - a (a - 1) / 2 + o
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int k = 0; k < NP; ++k) acc[j][k] = 0.0;
  int buf = 0;
  __syncthreads();  // the mode products
  for (int f = max(0, c0 + 1 - P); f <= c1; ++f) {  // f: index among all functions (0 is the boundary one)
    const int e = at[f];
    if (e >= 0) {
#pragma unroll 1
      for (int t0 = 0; t0 < Q; t0 += 2, buf ^= 1) {
        double* sv = sV + buf * 12 * kCol + lane;
        const int te = t0 + (mixed ? 1 : 0);
        if (te < Q) {
          const int q3 = __builtin_amdgcn_readfirstlane(e * Q + te);
          double x[3], J[3][3], v[7];
          column_eval(col, md.K, d3, sM, lane, q3, qx[q3], x, J);
          const double det = point_values<VAL_C>(g, x, J, w12 * qw[q3], v);
          if (!(det > 0.0)) *err = 1;
          double* o = sv + (mixed ? 6 * kCol : 0);
#pragma unroll
          for (int i = 0; i < 6; ++i) o[i * kCol] = v[i];
        }
        __syncthreads();  // two buffers: the next round writes the other one
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          if (t0 + d >= Q) break;
          // field j of the half: value v_j times first- and second-function factors
          // (B B, B B, B B, B' B') of C11, C12, C22, C33 or (B B', B' B) of C13 and C23
          const long long row = (long long)__builtin_amdgcn_readfirstlane(e * Q + t0 + d) * Q;
          ctab_t* B = val + row;
          ctab_t* Bd = der + row;
          ctab_t* X = (mixed ? der : val) + row;
          ctab_t* Y = (mixed ? val : der) + row;
          const double* __restrict__ vi = sv + 6 * d * kCol + (mixed ? 4 * kCol : 0);
          const double v0 = vi[0], v1 = mixed ? v0 : vi[kCol];
          const double v2 = vi[(mixed ? 1 : 2) * kCol], v3 = mixed ? v2 : vi[3 * kCol];
#pragma unroll
          for (int a = 0; a <= P; ++a) {
            const double u0 = v0 * B[a], u1 = v1 * X[a], u2 = v2 * B[a], u3 = v3 * Bd[a];
#pragma unroll
            for (int b = a; b <= P; ++b) {
              const int k = a * (P + 1) - a * (a - 1) / 2 + b - a;
              acc[0][k] = fma(u0, X[b], acc[0][k]);
              acc[1][k] = fma(u1, B[b], acc[1][k]);
              acc[2][k] = fma(u2, X[b], acc[2][k]);
              acc[3][k] = fma(u3, Y[b], acc[3][k]);
            }
          }
        }
      }
    }
    // function f is complete: store its pairs, move the others down by one
    if (f > c0 && live) {
      double* o = H + ((long long)(f - 1 - base) * (P + 1) * kFields3 + (mixed ? 4 : 0)) * nq12 + q12;
#pragma unroll
      for (int k = 0; k <= P; ++k)
        if (f - 1 + k < T.n[2]) {
#pragma unroll
          for (int j = 0; j < 4; ++j) o[(k * kFields3 + j) * nq12] = acc[j][k];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int a = 0; a < P; ++a)
#pragma unroll
        for (int o = 0; o <= P - a; ++o) {
          const int k = a * (P + 1) - a * (a - 1) / 2 + o;
          const int nx = (a + 1) * (P + 1) - (a + 1) * a / 2 + o;
          acc[j][k] = o < P - a ? acc[j][nx] : 0.0;
        }
      acc[j][NP - 1] = 0.0;
    }
  }
}

// Direction-3 moments M1[i3][ch][q2][q1] = sum over q3 of v_ch B_i3: the
// features' channels (NCH = kFeat) or w |det J| f of a load vector (NCH = 1).
// One thread per column and run of functions i3, walked as in k_contract3.
// Bound by the FP64 evaluation: 2.7 ms for the seven channels or the load vector
// at 112^3, p = 4.
template <int P, int NCH>
__global__ __launch_bounds__(kCol) void k_moment3(
    AcrossTables T, GeomDesc g, Modes md, RhsDesc rhs, int nq1, int nq2, cidx_t* at, ctab_t* qx, ctab_t* qw,
    ctab_t* val, ctab_t* d3, int base, int end, int len, double* __restrict__ M1) {
  extern __shared__ double sm[];
  constexpr int Q = P + 1;
  const long long nq12 = (long long)nq1 * nq2;
  const long long q12 = (long long)blockIdx.x * kCol + threadIdx.x;
  const int c0 = base + (int)blockIdx.y * len, c1 = min(c0 + len, end);
  if (q12 >= nq12 || c0 >= c1) return;
  const int q1 = (int)(q12 % nq1), q2 = (int)(q12 / nq1);
  const Column col = column_of(g, T.qx[0][q1], T.qx[1][q2]);
  column_modes(md, q1, q2, sm, threadIdx.x);
  const double w12 = T.qw[0][q1] * T.qw[1][q2];
  double acc[NCH][P + 1];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int a = 0; a <= P; ++a) acc[ch][a] = 0.0;
  for (int f = max(0, c0 + 1 - P); f <= c1; ++f) {
    const int e = at[f];
    if (e >= 0) {
#pragma unroll 1
      for (int t = 0; t < Q; ++t) {
        const int q3 = e * Q + t;
        const double w = w12 * qw[q3];
        double x[3], J[3][3], v[7];
        column_eval(col, md.K, d3, sm, threadIdx.x, q3, qx[q3], x, J);
        if constexpr (NCH == 1) {
          double A[3][3];
          v[0] = w * fabs(adjugate<3>(J, A)) * rhs_eval<3>(rhs, x);
        } else {
          point_values<VAL_FEAT>(g, x, J, w, v);
        }
#pragma unroll
        for (int a = 0; a <= P; ++a) {
          const double B = val[(long long)q3 * Q + a];
#pragma unroll
          for (int ch = 0; ch < NCH; ++ch) acc[ch][a] = fma(v[ch], B, acc[ch][a]);
        }
      }
    }
    if (f > c0) {
      double* o = M1 + (long long)(f - 1 - base) * NCH * nq12 + q12;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) o[ch * nq12] = acc[ch][0];
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
      for (int a = 0; a < P; ++a) acc[ch][a] = acc[ch][a + 1];
      acc[ch][P] = 0.0;
    }
  }
}

// Runs of direction-1 functions of k_contract12: 128 lanes cover
// the Gauss points of kRunElems elements, so of that many functions less p.
template <int P>
struct Run1 {
  static constexpr int Q = P + 1;
  static constexpr int ELEMS = 128 / Q;            // elements per run at most
  static constexpr int LEN = ELEMS - P;            // functions per run at most
  static constexpr int QP = Q | 1;                 // points of an element in LDS, odd: lanes one element apart
  static constexpr int QS = ELEMS * QP;            // fall on distinct banks
  static constexpr int TS = (Q * Q) | 1;           // (B, B') pairs of an element in LDS, odd for the same reason
  static int runs(int n) { return (n + LEN - 1) / LEN; }
  static int len(int n) { return (n + runs(n) - 1) / runs(n); }
};

typedef double d2_t __attribute__((ext_vector_type(2)));

// elements below the functions [f0, f1] (indices among all functions)
__device__ inline int first_elem(const int* at, int f0, int p) {
  int f = max(0, f0 - p);
  while (at[f] < 0) ++f;
  return at[f];
}
__device__ inline int last_elem(const int* at, int f1) {
  while (at[f1] < 0) --f1;
  return at[f1];
}

// v of the lane below (lane 0: 0), all lanes active
__device__ inline double wave_up1(double v) {
  union {
    double d;
    int i[2];
  } u;
  u.d = v;
  u.i[0] = __builtin_amdgcn_update_dpp(0, u.i[0], 0x138, 0xf, 0xf, true);  // wave_shr:1
  u.i[1] = __builtin_amdgcn_update_dpp(0, u.i[1], 0x138, 0xf, 0xf, true);
  return u.d;
}

// Directions 2 and 1, and the band.  Block (x: run of functions i1, y: pair
// (i3, i3 + o3), z: run of functions i2).  It walks the direction-2 functions:
// lane q of each half-block holds the Gauss column q1 of the run and, for the
// (p+1)^2 ordered pairs of the current element's functions, two of the four
// sums G_xy (x, y = 1: derivative in direction 1 on the first / second
// function), the first half G_11 and G_00 (one and four fields), the second
// G_10 and G_01 (three fields).  When the walk leaves function f, its 2p+1
// pairs of lines (rows f with columns f..f+p, rows f+1..f+p with column f) are
// complete and go to LDS.  Direction 1: a lane takes one line and one element
// (the one whose first function is f1), forms the element's (p+1)^2 local
// entries, and the entries of row i1 are gathered over the elements of its
// functions by shifting the local rows along the lanes (Horner's scheme in the
// shift); the 2p+1 band entries are stored, zeros where the column leaves the
// grid.
// Bound by the instruction issue of both contractions (two waves per SIMD at
// p = 4, 5): 112^3, p = 4: 7.5 ms in all.  A lane per row i1 that read the G of
// its elements from LDS took 10.6 ms (14 LDS reads per 14 FMAs); loading the next
// element's fields ahead gained nothing at p <= 4 and spilled at p = 5 (1343
// against 845 us per run of 72^3).
template <int P>
__global__ __launch_bounds__(2 * kCol, P <= 5 ? 2 : 1) void k_contract12(
    AcrossTables T, cidx_t* at, ctab_t* val, ctab_t* der, const double* __restrict__ H, double* __restrict__ band, long long Ns, int nq1, int nq2, int base, int len1,
    int len2) {
  extern __shared__ double sm[];
  using R = Run1<P>;
  constexpr int Q = R::Q, W = 2 * P + 1, NF = kFields3;
  constexpr int CENTER = (W * W * W - 1) / 2;
  constexpr int FX = 5;                           // fields read by the first half (the second: three)
  constexpr int LPW = 64 / R::ELEMS;              // lines per wave in direction 1
  double* sG = sm;                                          // [4][W][QS]
  d2_t* sT = reinterpret_cast<d2_t*>(sm + 4 * W * R::QS);   // [ELEMS][TS]
  const int tid = threadIdx.x;
  const int half = tid / kCol, q = tid % kCol;
  const int n1 = T.n[0], n2 = T.n[1], n3 = T.n[2];
  const int s0 = (int)blockIdx.x * len1, s1 = min(s0 + len1, n1);
  const int g0 = (int)blockIdx.z * len2, g1 = min(g0 + len2, n2);
  const int pair = (int)blockIdx.y;
  const int o3 = pair % (P + 1), i3 = base + pair / (P + 1);
  if (s0 >= s1 || g0 >= g1) return;
  const bool in3 = i3 + o3 < n3;
  const int elo = first_elem(T.at[0], s0 + 1, P), ehi = last_elem(T.at[0], s1);
  const int nE = ehi - elo + 1;
  for (int k = tid; k < nE * Q * Q; k += 2 * kCol) {
    const int e = k / (Q * Q), r = k % (Q * Q);
    sT[e * R::TS + r] = d2_t{T.val[0][(long long)(elo + e) * Q * Q + r], T.der[0][(long long)(elo + e) * Q * Q + r]};
  }
  const bool live = in3 && q < nE * Q;
  const long long nq12 = (long long)nq1 * nq2;
  const double* __restrict__ Hc = H + (long long)pair * NF * nq12 + elo * Q + (live ? q : 0);
  const int slot = (q / Q) * R::QP + q % Q;
  // direction 1: this lane's line of a wave's LPW and its element (first function s0 + 1 - P + j)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = lane / R::ELEMS, j = lane % R::ELEMS;
  const int nl = s1 - s0;
  const bool on = sub < LPW && j < nl + P;
  const int f1 = s0 + 1 - P + j;
  int el = on && f1 >= 0 ? T.at[0][f1] : -1;
  el = el < 0 ? -1 : el - elo;
  const int i1 = f1 - 1;  // the row the lane holds after the shifts (j >= P)
  double ga[P + 1][P + 1], gb[P + 1][P + 1];
#pragma unroll
  for (int a = 0; a <= P; ++a)
#pragma unroll
    for (int b = 0; b <= P; ++b) ga[a][b] = gb[a][b] = 0.0;
  // fields of the first half: 11, 32, 33, 22, 23; of the second: 31, 12, 13 and zeros
  const long long off[3] = {half == 0 ? 0 : 5 * nq12, half == 0 ? 7 * nq12 : nq12, half == 0 ? 3 * nq12 : 4 * nq12};
  double hq[Q][FX];
#pragma unroll
  for (int t = 0; t < Q; ++t)
#pragma unroll
    for (int k = 0; k < FX; ++k) hq[t][k] = 0.0;
  auto load = [&](int e, int t, double (&h)[FX]) {
    const double* __restrict__ p = Hc + ((long long)e * Q + t) * nq1;
#pragma unroll
    for (int k = 0; k < 3; ++k) h[k] = p[off[k]];
    if (half == 0) {
      h[3] = p[2 * nq12];
      h[4] = p[6 * nq12];
    }
  };
  for (int f = g0 + 1 - P; f <= g1; ++f) {
    const int e = f >= 0 ? at[f] : -1;
    if (e >= 0 && live) {
#pragma unroll
      for (int t = 0; t < Q; ++t) load(e, t, hq[t]);
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const double(&h)[FX] = hq[t];
        ctab_t* B = val + ((long long)e * Q + t) * Q;
        ctab_t* Bd = der + ((long long)e * Q + t) * Q;
        // ga: G_11 | G_01, gb: G_00 | G_10; the terms a half does not have are zero
        const double h12 = half == 0 ? 0.0 : h[1];
#pragma unroll
        for (int a = 0; a <= P; ++a) {
          const double u = fma(h12, Bd[a], h[0] * B[a]);
          const double ud = fma(h[3], Bd[a], h[1] * B[a]), ub = fma(h[4], Bd[a], h[2] * B[a]);
#pragma unroll
          for (int b = 0; b <= P; ++b) {
            ga[a][b] = fma(u, B[b], ga[a][b]);
            gb[a][b] = fma(ud, Bd[b], fma(ub, B[b], gb[a][b]));
          }
        }
      }
    }
    // lines (row, column) completed by leaving f: slot l = o2 + P
    __syncthreads();  // the previous lines have been read
    if (live) {
      double* o0 = sG + (half == 0 ? 0 : 2) * (W * R::QS) + slot;
      double* o1 = sG + (half == 0 ? 3 : 1) * (W * R::QS) + slot;
#pragma unroll
      for (int k = 0; k <= P; ++k) {
        o0[(P + k) * R::QS] = ga[0][k];
        o1[(P + k) * R::QS] = gb[0][k];
        if (k > 0) {
          o0[(P - k) * R::QS] = ga[k][0];
          o1[(P - k) * R::QS] = gb[k][0];
        }
      }
    }
#pragma unroll
    for (int a = 0; a <= P; ++a)
#pragma unroll
      for (int b = 0; b <= P; ++b) {
        ga[a][b] = a < P && b < P ? ga[a < P ? a + 1 : P][b < P ? b + 1 : P] : 0.0;
        gb[a][b] = a < P && b < P ? gb[a < P ? a + 1 : P][b < P ? b + 1 : P] : 0.0;
      }
    __syncthreads();
    // the groups of LPW lines, dealt to the four waves from a start that moves with f
    for (int task = (wave + f + P) & 3; task * LPW < W; task += 4) {
      const int l = task * LPW + sub;
      const int o2 = l - P;
      const int i2 = (o2 >= 0 ? f : f - o2) - 1, j2 = i2 + o2;
      const bool mine = on && l < W && i2 >= g0 && i2 < g1 && !(o3 == 0 && o2 < 0);
      if (__ballot(mine) == 0) continue;
      const bool in = in3 && j2 >= 0 && j2 < n2;
      double lc[P + 1][P + 1];
#pragma unroll
      for (int a = 0; a <= P; ++a)
#pragma unroll
        for (int b = 0; b <= P; ++b) lc[a][b] = 0.0;
      if (mine && in && el >= 0) {
        const d2_t* __restrict__ tb = sT + el * R::TS;
        const double* __restrict__ G = sG + l * R::QS + el * R::QP;
#pragma unroll 1
        for (int t = 0; t < Q; ++t, tb += Q, ++G) {
          const double g11 = G[0], g10 = G[W * R::QS], g01 = G[2 * W * R::QS], g00 = G[3 * W * R::QS];
          d2_t bb[P + 1];
#pragma unroll
          for (int b = 0; b <= P; ++b) bb[b] = tb[b];
#pragma unroll
          for (int a = 0; a <= P; ++a) {
            const double u = fma(g11, bb[a].y, g01 * bb[a].x);
            const double v = fma(g10, bb[a].y, g00 * bb[a].x);
#pragma unroll
            for (int b = 0; b <= P; ++b) lc[a][b] = fma(u, bb[b].y, fma(v, bb[b].x, lc[a][b]));
          }
        }
      }
      // row i1, column i1 + o: the sum over a of the local entry (a, a + o) of
      // the element whose first function lies a below i1, a lanes down
      double s[W];
#pragma unroll
      for (int o = 0; o < W; ++o) s[o] = 0.0;
#pragma unroll
      for (int a = P; a >= 0; --a) {
#pragma unroll
        for (int o = 0; o < W; ++o) {  // offset o - P: rows a+1..P reach from -P to P - a - 1
          if (a < P && o <= 2 * P - a - 1) s[o] = wave_up1(s[o]);
          if (o >= P - a && o <= 2 * P - a) s[o] += lc[a][o - P + a >= 0 && o - P + a <= P ? o - P + a : 0];
        }
      }
      if (!mine || j < P) continue;
      double* __restrict__ row = band + i1 + (long long)n1 * (i2 + (long long)n2 * i3);
      const int p0 = ((o3 + P) * W + l) * W - CENTER;
#pragma unroll
      for (int o = 0; o < W; ++o) {
        const int j1 = i1 + o - P;
        if (o3 == 0 && o2 == 0 && o < P) continue;
        row[(long long)(p0 + o) * Ns] = j1 >= 0 && j1 < n1 ? s[o] : 0.0;
      }
    }
  }
}

// Moments, direction 2: M2[i3][ch][i2][q1] from M1[i3][ch][q2][q1]; one thread
// per (q1, channel plane y) and run of functions i2.
template <int P>
__global__ __launch_bounds__(kCol) void k_moment2(AcrossTables T, cidx_t* at,
                                                  ctab_t* val, const double* __restrict__ M1,
                                                  double* __restrict__ M2, int nq1, int nq2, int len2) {
  constexpr int Q = P + 1;
  const int q1 = (int)blockIdx.x * kCol + threadIdx.x;
  const int n2 = T.n[1], g0 = (int)blockIdx.z * len2, g1 = min(g0 + len2, n2);
  if (q1 >= nq1 || g0 >= g1) return;
  const double* __restrict__ in = M1 + (long long)blockIdx.y * nq1 * nq2 + q1;
  double* __restrict__ out = M2 + (long long)blockIdx.y * nq1 * n2 + q1;
  double acc[P + 1];
#pragma unroll
  for (int a = 0; a <= P; ++a) acc[a] = 0.0;
  for (int f = max(0, g0 + 1 - P); f <= g1; ++f) {
    const int e = at[f];
    if (e >= 0) {
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const long long q2 = (long long)e * Q + t;
        const double v = in[q2 * nq1];
#pragma unroll
        for (int a = 0; a <= P; ++a) acc[a] = fma(v, val[q2 * Q + a], acc[a]);
      }
    }
    if (f > g0) out[(long long)(f - 1) * nq1] = acc[0];
#pragma unroll
    for (int a = 0; a < P; ++a) acc[a] = acc[a + 1];
    acc[P] = 0.0;
  }
}

// sum_t w_t B_i(t) of direction l and function i (0-based interior index)
template <int P>
__device__ inline double moment1(const AcrossTables& T, int l, int i) {
  constexpr int Q = P + 1;
  double s = 0.0;
#pragma unroll
  for (int a = 0; a <= P; ++a) {
    const int e = i + 1 - a >= 0 ? T.at[l][i + 1 - a] : -1;
    if (e < 0) continue;
#pragma unroll
    for (int t = 0; t < Q; ++t) s = fma(T.qw[l][e * Q + t], T.val[l][(e * Q + t) * Q + a], s);
  }
  return s;
}

// Moments, direction 1, for the planes i3 of [base, end), one thread per dof:
// b_i (NCH = 1), or the features feat_i = (M_ch / M_w, p) in FP32, the moment
// of w a product of univariate ones.
template <int P, int NCH, typename Out>
__global__ __launch_bounds__(kBlock) void k_moment1(AcrossTables T, const double* __restrict__ M2, int nq1, int base,
                                                    int end, Out* __restrict__ out) {
  constexpr int Q = P + 1;
  const int n1 = T.n[0], n2 = T.n[1];
  const long long k = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (k >= (long long)n1 * n2 * (end - base)) return;
  const int i1 = (int)(k % n1);
  const long long r = k / n1;
  const int i2 = (int)(r % n2), i3 = (int)(r / n2);  // i3 relative to base
  double s[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) s[ch] = 0.0;
#pragma unroll
  for (int a = 0; a <= P; ++a) {
    const int e = i1 + 1 - a >= 0 ? T.at[0][i1 + 1 - a] : -1;
    if (e < 0) continue;
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const double B = T.val[0][(e * Q + t) * Q + a];
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        s[ch] = fma(B, M2[(((long long)i3 * NCH + ch) * n2 + i2) * nq1 + e * Q + t], s[ch]);
    }
  }
  const long long row = i1 + (long long)n1 * (i2 + (long long)n2 * (base + i3));
  if constexpr (NCH == 1) {
    out[row] = s[0];
  } else {
    const double den = moment1<P>(T, 0, i1) * moment1<P>(T, 1, i2) * moment1<P>(T, 2, base + i3);
    const double inv = 1.0 / den;
    typedef float f4_t __attribute__((ext_vector_type(4)));
    f4_t* o = reinterpret_cast<f4_t*>(out + 8 * row);
    o[0] = f4_t{(float)(s[0] * inv), (float)(s[1] * inv), (float)(s[2] * inv), (float)(s[3] * inv)};
    o[1] = f4_t{(float)(s[4] * inv), (float)(s[5] * inv), (float)(s[6] * inv), (float)P};
  }
}

// b_i += sum_t w_t |det J| f(F(t)) B_i(t) over one colour class of elements.
template <int D, int P>
__global__ __launch_bounds__(kBlock) void k_load(Tables T, GeomDesc g, RhsDesc rhs, double* __restrict__ b,
                                                 int c1, int c2, int c3, int m1, int m2) {
  constexpr int Q = P + 1, L = P + 1;
  constexpr int Q3 = (D == 3) ? Q : 1;
  constexpr int L3 = (D == 3) ? L : 1;
  constexpr int NQ = Q * Q * Q3;
  __shared__ double sg[NQ];
  __shared__ double sV[3][Q][L];
  int bid = blockIdx.x;
  const int j1 = bid % m1;
  bid /= m1;
  const int j2 = bid % m2;
  const int j3 = bid / m2;
  const int e[3] = {c1 + j1 * (P + 1), c2 + j2 * (P + 1), (D == 3) ? c3 + j3 * (P + 1) : 0};
  const int tid = threadIdx.x;
  for (int idx = tid; idx < 3 * Q * L; idx += kBlock) {
    const int l = idx / (Q * L), t = (idx / L) % Q, a = idx % L;
    sV[l][t][a] = (l < D) ? T.val[l][(e[l] * Q + t) * L + a] : ((t == 0 && a == 0) ? 1.0 : 0.0);
  }
  for (int t = tid; t < NQ; t += kBlock) {
    const int t1 = t % Q, t2 = (t / Q) % Q, t3 = t / (Q * Q);
    double xi[3] = {T.qx[0][e[0] * Q + t1], T.qx[1][e[1] * Q + t2], 0.0};
    double w = T.qw[0][e[0] * Q + t1] * T.qw[1][e[1] * Q + t2];
    if (D == 3) {
      xi[2] = T.qx[2][e[2] * Q + t3];
      w *= T.qw[2][e[2] * Q + t3];
    }
    double x[3], J[3][3], A[3][3];
    map_eval<D>(g, xi, x, J);
    const double det = adjugate<D>(J, A);
    sg[t] = w * fabs(det) * rhs_eval<D>(rhs, x);
  }
  __syncthreads();
  for (int idx = tid; idx < L * L * L3; idx += kBlock) {
    const int a1 = idx % L, a2 = (idx / L) % L, a3 = idx / (L * L);
    const int r1 = T.first[0][e[0]] + a1 - 1, r2 = T.first[1][e[1]] + a2 - 1;
    const int r3 = (D == 3) ? T.first[2][e[2]] + a3 - 1 : 0;
    if (r1 < 0 || r1 >= T.n[0] || r2 < 0 || r2 >= T.n[1] || r3 < 0 || r3 >= T.n[2]) continue;
    double s = 0.0;
    for (int t = 0; t < NQ; ++t) {
      const int t1 = t % Q, t2 = (t / Q) % Q, t3 = t / (Q * Q);
      s += sg[t] * sV[0][t1][a1] * sV[1][t2][a2] * sV[2][t3][a3];
    }
    b[r1 + (long long)T.n[0] * (r2 + (long long)T.n[1] * r3)] += s;
  }
}

// Per-dof geometry/coefficient statistics for the learned scaling, without
// assembling A: the same Gauss-point values as k_assemble's feature channels
// (w G's six entries, w kappa, w), summed into acc by feature_sums.
template <int D, int P>
__global__ __launch_bounds__(kBlock) void k_features(Tables T, GeomDesc g, double* __restrict__ acc, int c1, int c2,
                                                     int c3, int m1, int m2) {
  constexpr int Q = P + 1, L = P + 1;
  constexpr int Q3 = (D == 3) ? Q : 1;
  constexpr int NQ = Q * Q * Q3;
  __shared__ double sf[8][NQ];
  __shared__ double sV[3][Q][L];
  __shared__ double sF1[8 * L * Q * Q3], sF2[8 * L * L * Q3];
  __shared__ int sFirst[3];
  int bid = blockIdx.x;
  const int j1 = bid % m1;
  bid /= m1;
  const int j2 = bid % m2;
  const int j3 = bid / m2;
  const int e[3] = {c1 + j1 * (P + 1), c2 + j2 * (P + 1), (D == 3) ? c3 + j3 * (P + 1) : 0};
  const int tid = threadIdx.x;
  for (int idx = tid; idx < 3 * Q * L; idx += kBlock) {
    const int l = idx / (Q * L), t = (idx / L) % Q, a = idx % L;
    sV[l][t][a] = (l < D) ? T.val[l][(e[l] * Q + t) * L + a] : ((t == 0 && a == 0) ? 1.0 : 0.0);
  }
  if (tid < 3) sFirst[tid] = (tid < D) ? T.first[tid][e[tid]] : 1;
  for (int t = tid; t < NQ; t += kBlock) {
    const int t1 = t % Q, t2 = (t / Q) % Q, t3 = t / (Q * Q);
    double xi[3] = {T.qx[0][e[0] * Q + t1], T.qx[1][e[1] * Q + t2], 0.0};
    double w = T.qw[0][e[0] * Q + t1] * T.qw[1][e[1] * Q + t2];
    if (D == 3) {
      xi[2] = T.qx[2][e[2] * Q + t3];
      w *= T.qw[2][e[2] * Q + t3];
    }
    double x[3], J[3][3], A[3][3] = {};
    map_eval<D>(g, xi, x, J);
    const double det = fabs(adjugate<D>(J, A));
    double G[3][3];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) {
        double s = 0.0;
        for (int k = 0; k < D; ++k) s += A[a][k] * A[b][k];
        G[a][b] = (a < D && b < D) ? s / det : 0.0;
      }
    sf[0][t] = w * G[0][0];
    sf[1][t] = w * G[1][1];
    sf[2][t] = w * G[2][2];
    sf[3][t] = w * G[0][1];
    sf[4][t] = w * G[0][2];
    sf[5][t] = w * G[1][2];
    sf[6][t] = w * kappa_eval(g, x);
    sf[7][t] = w;
  }
  __syncthreads();
  feature_sums<D, P>(&sf[0][0], sV, sFirst, T, sF1, sF2, acc);
}

// Extreme eigenvalues of a symmetric positive definite 2x2 / 3x3 matrix.
// 2x2: closed form, the small one as det / large (no cancellation).  3x3:
// cyclic Jacobi rotations (each zeroes one off-diagonal pair; the diagonal
// converges quadratically to the eigenvalues, accurate to roundoff also for
// repeated eigenvalues, where closed forms of the cubic lose half the digits).
__device__ inline void sym_extremes(int d, const double Q[3][3], double& lo, double& hi) {
  if (d == 2) {
    const double m = 0.5 * (Q[0][0] + Q[1][1]), h = 0.5 * (Q[0][0] - Q[1][1]);
    hi = m + sqrt(h * h + Q[0][1] * Q[0][1]);
    lo = (Q[0][0] * Q[1][1] - Q[0][1] * Q[0][1]) / hi;
    return;
  }
  double a[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) a[i][j] = Q[i][j];
  for (int sweep = 0; sweep < 12; ++sweep) {
    const double off = a[0][1] * a[0][1] + a[0][2] * a[0][2] + a[1][2] * a[1][2];
    const double dia = a[0][0] * a[0][0] + a[1][1] * a[1][1] + a[2][2] * a[2][2];
    if (off <= 1e-36 * dia) break;
    for (int k = 0; k < 3; ++k) {
      const int p = k == 2 ? 1 : 0, q = k == 0 ? 1 : 2;
      const double apq = a[p][q];
      if (fabs(apq) <= 1e-300) continue;
      // rotation angle with tan(2 phi) = 2 a_pq / (a_qq - a_pp); t = tan(phi), the smaller root
      const double theta = (a[q][q] - a[p][p]) / (2.0 * apq);
      const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
      const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
      a[p][p] -= t * apq;
      a[q][q] += t * apq;
      a[p][q] = a[q][p] = 0.0;
      const int r = 3 - p - q;
      const double arp = a[r][p], arq = a[r][q];
      a[r][p] = a[p][r] = c * arp - s * arq;
      a[r][q] = a[q][r] = s * arp + c * arq;
    }
  }
  lo = fmin(a[0][0], fmin(a[1][1], a[2][2]));
  hi = fmax(a[0][0], fmax(a[1][1], a[2][2]));
}

// min / max over the Gauss points of the extreme eigenvalues of
// Q = kappa |det J| J^-1 J^-T (Sec. 2.1 eq. Q), and the max over the points of
// the local ratio lambda_max(Q(x)) / lambda_min(Q(x)).  Grid-stride over all
// points (nq[l] = points along direction l, flat index i1 + nq0 (i2 + nq1 i3));
// per block part[blockIdx.x] = min, part[G + blockIdx.x] = max and
// part[2 G + blockIdx.x] = max ratio (G = gridDim.x).
template <int D>
__global__ __launch_bounds__(kBlock) void k_qbounds(const double* __restrict__ qx0, const double* __restrict__ qx1,
                                                    const double* __restrict__ qx2, GeomDesc g, int nq0, int nq1,
                                                    int nq2, double* __restrict__ part) {
  double lo = INFINITY, hi = -INFINITY, loc = 0.0;
  const long long total = (long long)nq0 * nq1 * nq2;
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < total; i += (long long)gridDim.x * kBlock) {
    const int i1 = (int)(i % nq0);
    const long long rest = i / nq0;
    const int i2 = (int)(rest % nq1), i3 = (int)(rest / nq1);
    const double xi[3] = {qx0[i1], qx1[i2], D == 3 ? qx2[i3] : 0.0};
    double x[3], J[3][3], A[3][3] = {};
    map_eval<D>(g, xi, x, J);
    const double det = fabs(adjugate<D>(J, A));
    const double k = kappa_eval(g, x) / det;
    double Q[3][3];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) {
        double s = 0.0;
        for (int l = 0; l < D; ++l) s += A[a][l] * A[b][l];
        Q[a][b] = k * s;
      }
    double l0, l1;
    sym_extremes(D, Q, l0, l1);
    lo = fmin(lo, l0);
    hi = fmax(hi, l1);
    loc = fmax(loc, l1 / l0);
  }
  // min / max are exact: any reduction order gives the same result
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_down(lo, off, 64));
    hi = fmax(hi, __shfl_down(hi, off, 64));
    loc = fmax(loc, __shfl_down(loc, off, 64));
  }
  __shared__ double slo[kBlock / 64], shi[kBlock / 64], sloc[kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    slo[wid] = lo;
    shi[wid] = hi;
    sloc[wid] = loc;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) {
      lo = fmin(lo, slo[w]);
      hi = fmax(hi, shi[w]);
      loc = fmax(loc, sloc[w]);
    }
    part[blockIdx.x] = lo;
    part[gridDim.x + blockIdx.x] = hi;
    part[2 * gridDim.x + blockIdx.x] = loc;
  }
}

__global__ void k_minmax(const double* __restrict__ part, int count, double* __restrict__ out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double lo = INFINITY, hi = -INFINITY, loc = 0.0;
  for (int k = 0; k < count; ++k) {
    lo = fmin(lo, part[k]);
    hi = fmax(hi, part[count + k]);
    loc = fmax(loc, part[2 * count + k]);
  }
  out[0] = lo;
  out[1] = hi;
  out[2] = loc;
}

// feat[i] = (acc[i][0..6] / acc[i][7], p) in FP32
__global__ void k_features_finish(const double* __restrict__ acc, float* __restrict__ feat, long long N, int p) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const double inv = 1.0 / acc[8 * i + 7];
  for (int ch = 0; ch < 7; ++ch) feat[8 * i + ch] = (float)(acc[8 * i + ch] * inv);
  feat[8 * i + 7] = (float)p;
}

// diag(P)_i = sum_j K_j[i_j, i_j] prod_{l != j} M_l[i_l, i_l]  (Sec. 3 Kronecker sum)
__device__ inline double diagP_at(const double* m1, const double* k1, const double* m2, const double* k2,
                                  const double* m3, const double* k3, int n1, int n2, int dim, long long i) {
  const int i1 = (int)(i % n1);
  const long long t = i / n1;
  const int i2 = (int)(t % n2), i3 = (int)(t / n2);
  if (dim == 2) return k1[i1] * m2[i2] + m1[i1] * k2[i2];
  return k1[i1] * m2[i2] * m3[i3] + m1[i1] * k2[i2] * m3[i3] + m1[i1] * m2[i2] * k3[i3];
}

__global__ void k_diagP(const double* m1, const double* k1, const double* m2, const double* k2,
                        const double* m3, const double* k3, int n1, int n2, long long N, int dim,
                        double* out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) out[i] = diagP_at(m1, k1, m2, k2, m3, k3, n1, n2, dim, i);
}

// a fill kernel instead of a memset: callers may capture these launches into graphs
__global__ void k_zero(double* __restrict__ p, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0.0;
}

__global__ void k_copy_plane(const double* __restrict__ src, double* __restrict__ dst, long long N) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < N) dst[i] = src[i];
}

Tables make_tables(const igafd_ctx* c) {
  Tables T{};
  for (int l = 0; l < 3; ++l) {
    T.first[l] = c->ddir[l].elem_first;
    T.qx[l] = c->ddir[l].qx;
    T.qw[l] = c->ddir[l].qw;
    T.val[l] = c->ddir[l].val;
    T.der[l] = c->ddir[l].der;
    T.n[l] = c->n[l];
  }
  return T;
}

AcrossTables across_tables(const igafd_ctx* c) {
  AcrossTables T{};
  static_cast<Tables&>(T) = make_tables(c);
  for (int l = 0; l < 3; ++l) T.at[l] = c->ddir[l].elem_at;
  return T;
}

int mode_count(const igafd_ctx* c) {  // padded
  return c->geom.kind == IGAFD_GEOM_WARPED ? (c->geom.nmodes + kModePad - 1) / kModePad * kModePad : 0;
}

Modes modes_of(const igafd_ctx* c) {
  Modes m{};
  m.K = mode_count(c);
  m.d12[0] = c->modes;
  m.d12[1] = m.d12[0] + 2LL * c->dir[0].nel * c->dir[0].q * m.K;
  m.d3 = m.d12[1] + 2LL * c->dir[1].nel * c->dir[1].q * m.K;
  return m;
}

int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

constexpr long long kAsmWorkMax = 2LL << 30;  // bytes of the direction-3 contraction kept at a time
constexpr int kAsmBlocks = 2048;              // blocks that fill the chip (256 CUs, several blocks each)

size_t mode_lds(int K) { return sizeof(double) * 3 * (size_t)K * kCol; }

// functions i3 per thread of the column kernels over `count` of them: long
// runs repeat less of the evaluation, short ones fill the chip
int column_run(int count, int colb) { return std::min(count, std::max(2, cdiv((long long)count * colb, kAsmBlocks))); }

// moments of directions 2 and 1 for the planes [base, end): M1 -> M2 -> out
template <int P, int NCH, typename Out>
igafd_status moments21(igafd_ctx* c, const AcrossTables& T, const double* M1, double* M2, int base, int end, Out* out) {
  const int nq1 = c->dir[0].nel * (P + 1), nq2 = c->dir[1].nel * (P + 1), n2 = c->n[1];
  const int planes = (end - base) * NCH, qb = cdiv(nq1, kCol);
  const int len2 = std::min(n2, std::max(4, cdiv(n2, cdiv(kAsmBlocks, (long long)qb * planes))));
  hipLaunchKernelGGL((k_moment2<P>), dim3((unsigned)qb, (unsigned)planes, (unsigned)cdiv(n2, len2)), dim3(kCol), 0,
                     c->stream, T, (cidx_t*)T.at[1], (ctab_t*)T.val[1], M1, M2, nq1, nq2, len2);
  hipLaunchKernelGGL((k_moment1<P, NCH, Out>), dim3((unsigned)cdiv((long long)c->n[0] * n2 * (end - base), kBlock)),
                     dim3(kBlock), 0, c->stream, T, M2, nq1, base, end, out);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

// Assembly of the band and the features across the elements, through a workspace of direction-3
// contractions for a run of planes i3 at a time: every further run repeats the
// evaluation of p element layers, so the run is as long as half the band's own
// bytes (at most kAsmWorkMax) allow; it is halved when that much memory is not
// there, down to one plane.
template <int P>
igafd_status launch_across(igafd_ctx* c, AsmWork* work) {
  using R = Run1<P>;
  constexpr int W = 2 * P + 1, NP3 = P + 1, NF = kFields3;
  const AcrossTables T = across_tables(c);
  const int nq1 = c->dir[0].nel * R::Q, nq2 = c->dir[1].nel * R::Q;
  const int n2 = c->n[1], n3 = c->n[2];
  const long long nq12 = (long long)nq1 * nq2;
  const long long layer = std::max((long long)NP3 * NF * nq12, kFeat * (nq12 + (long long)n2 * nq1));
  const long long cap = std::min(kAsmWorkMax, (long long)sizeof(double) * c->H * c->Ns / 2);
  int run = (int)std::max(1LL, std::min((long long)n3, cap / (layer * (long long)sizeof(double))));
  run = cdiv(n3, cdiv(n3, run));
  igafd_status st;
  while ((st = block_alloc((void**)&work->ws, sizeof(double) * (size_t)run * (size_t)layer)) != IGAFD_OK) {
    if (run == 1) return st;
    run = (run + 1) / 2;
  }
  double* ws = work->ws;
  // the zero halo of every plane; the rows in between are all written below
  const size_t pitch = sizeof(double) * (size_t)c->Ns;
  const long long tail = c->halo + c->N;
  IGAFD_HIP_CHECK(hipMemset2DAsync(c->band, pitch, 0, sizeof(double) * (size_t)c->halo, c->H, c->stream));
  IGAFD_HIP_CHECK(
      hipMemset2DAsync(c->band + tail, pitch, 0, sizeof(double) * (size_t)(c->Ns - tail), c->H, c->stream));
  const Modes md = modes_of(c);
  const size_t col_lds = mode_lds(md.K), lds3 = col_lds + sizeof(double) * 24 * kCol;
  // the limit of the function for any problem, not for this one's modes: another
  // thread's setup of the same degree may be between its setting and its launch
  constexpr int lds3_max = (int)(sizeof(double) * (3 * kMaxModes + 24) * kCol);
  static_assert(kMaxModes % kModePad == 0, "padded modes beyond kMaxModes");
  const int colb = cdiv(nq12, kCol);
  const size_t lds = sizeof(double) * (4 * W * R::QS + 2 * R::ELEMS * R::TS);
  IGAFD_HIP_CHECK(
      hipFuncSetAttribute((const void*)k_contract12<P>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  IGAFD_HIP_CHECK(
      hipFuncSetAttribute((const void*)k_contract3<P>, hipFuncAttributeMaxDynamicSharedMemorySize, lds3_max));
  const int runs1 = R::runs(c->n[0]), len1 = R::len(c->n[0]);
  for (int base = 0; base < n3; base += run) {
    const int end = std::min(n3, base + run);
    const int len = column_run(end - base, colb);
    hipLaunchKernelGGL((k_contract3<P>), dim3((unsigned)colb, (unsigned)cdiv(end - base, len)), dim3(2 * kCol), lds3,
                       c->stream, T, c->geom, md, nq1, nq2, (cidx_t*)T.at[2], (ctab_t*)T.qx[2],
                       (ctab_t*)T.qw[2], (ctab_t*)T.val[2], (ctab_t*)T.der[2], (ctab_t*)md.d3, base, end,
                       len, ws, c->dflag);
    IGAFD_HIP_CHECK(hipGetLastError());
    const int pairs = (end - base) * NP3;
    const int len2 = std::min(n2, std::max(4, cdiv(n2, cdiv(kAsmBlocks / 2, (long long)runs1 * pairs))));
    hipLaunchKernelGGL((k_contract12<P>), dim3((unsigned)runs1, (unsigned)pairs, (unsigned)cdiv(n2, len2)),
                       dim3(2 * kCol), lds, c->stream, T, (cidx_t*)T.at[1], (ctab_t*)T.val[1], (ctab_t*)T.der[1], ws, c->band + c->halo, c->Ns, nq1, nq2, base, len1, len2);
    IGAFD_HIP_CHECK(hipGetLastError());
  }
  for (int base = 0; base < n3; base += run) {
    const int end = std::min(n3, base + run);
    const int len = column_run(end - base, colb);
    hipLaunchKernelGGL((k_moment3<P, kFeat>), dim3((unsigned)colb, (unsigned)cdiv(end - base, len)), dim3(kCol),
                       col_lds, c->stream, T, c->geom, md, RhsDesc{}, nq1, nq2, (cidx_t*)T.at[2], (ctab_t*)T.qx[2],
                       (ctab_t*)T.qw[2], (ctab_t*)T.val[2], (ctab_t*)md.d3,
                       base, end, len, ws);
    IGAFD_HIP_CHECK(hipGetLastError());
    st = moments21<P, kFeat>(c, T, ws, ws + (long long)(end - base) * kFeat * nq12, base, end, c->feat);
    if (st != IGAFD_OK) return st;
  }
  return IGAFD_OK;
}

// Load vector across the elements, through the moments of a run of planes i3 at
// a time, held in the context's CG vectors; nothing is allocated.
template <int P>
igafd_status load_across(igafd_ctx* c, RhsDesc rhs, double* b) {
  using R = Run1<P>;
  const AcrossTables T = across_tables(c);
  const Modes md = modes_of(c);
  const int nq1 = c->dir[0].nel * R::Q, nq2 = c->dir[1].nel * R::Q, n2 = c->n[1], n3 = c->n[2];
  const int colb = cdiv((long long)nq1 * nq2, kCol);
  const long long nq12 = (long long)nq1 * nq2, layer = nq12 + (long long)n2 * nq1;
  const int run = (int)std::min((long long)n3, c->scratch_len / layer);
  if (run < 1) {
    set_error("internal: scratch smaller than one plane of moments");
    return IGAFD_ERR_ARG;
  }
  for (int base = 0; base < n3; base += run) {
    const int end = std::min(n3, base + run);
    const int len = column_run(end - base, colb);
    hipLaunchKernelGGL((k_moment3<P, 1>), dim3((unsigned)colb, (unsigned)cdiv(end - base, len)), dim3(kCol),
                       mode_lds(md.K), c->stream, T, c->geom, md, rhs, nq1, nq2, (cidx_t*)T.at[2], (ctab_t*)T.qx[2],
                       (ctab_t*)T.qw[2], (ctab_t*)T.val[2], (ctab_t*)md.d3, base, end, len, c->scratch);
    const igafd_status st = moments21<P, 1>(c, T, c->scratch, c->scratch + (end - base) * nq12, base, end, b);
    if (st != IGAFD_OK) return st;
  }
  return IGAFD_OK;
}

template <int D, int P>
igafd_status launch_elements(igafd_ctx* c, double* acc) {
  const Tables T = make_tables(c);
  const int nel[3] = {c->ddir[0].nel, c->ddir[1].nel, D == 3 ? c->ddir[2].nel : 1};
  const int C3 = (D == 3) ? P + 1 : 1;
  for (int c3 = 0; c3 < C3; ++c3)
    for (int c2 = 0; c2 <= P; ++c2)
      for (int c1 = 0; c1 <= P; ++c1) {
        const int m1 = c1 < nel[0] ? (nel[0] - c1 + P) / (P + 1) : 0;
        const int m2 = c2 < nel[1] ? (nel[1] - c2 + P) / (P + 1) : 0;
        const int m3 = (D == 3) ? (c3 < nel[2] ? (nel[2] - c3 + P) / (P + 1) : 0) : 1;
        const long long blocks = (long long)m1 * m2 * m3;
        if (blocks == 0) continue;
        if (D == 2 && acc)
          hipLaunchKernelGGL((k_assemble<2, P, 1>), dim3((unsigned)blocks), dim3(kBlock), 0, c->stream, T, c->geom,
                             c->band + c->halo, c->Ns, c1, c2, c3, m1, m2, c->dflag, acc);
        else
          hipLaunchKernelGGL((k_assemble<D, P, 0>), dim3((unsigned)blocks), dim3(kBlock), 0, c->stream, T, c->geom,
                             c->band + c->halo, c->Ns, c1, c2, c3, m1, m2, c->dflag, nullptr);
        IGAFD_HIP_CHECK(hipGetLastError());
      }
  return IGAFD_OK;
}

// A's band and, when asked for, the features: across the elements in 3D with
// features, element by element otherwise (see the head of this file).
template <int D, int P>
igafd_status launch_assemble(igafd_ctx* c, bool with_features, AsmWork* work) {
  if (D == 3 && with_features) return launch_across<P>(c, work);
  IGAFD_HIP_CHECK(hipMemsetAsync(c->band, 0, sizeof(double) * c->H * c->Ns, c->stream));
  double* acc = nullptr;
  igafd_status st;
  if (with_features) {  // feature sums (8 per dof) assembled with A, kept as FP32 features
    if ((st = block_alloc((void**)&work->ws, sizeof(double) * 8 * (size_t)c->N)) != IGAFD_OK) return st;
    acc = work->ws;
    IGAFD_HIP_CHECK(hipMemsetAsync(acc, 0, sizeof(double) * 8 * (size_t)c->N, c->stream));
  }
  if ((st = launch_elements<D, P>(c, acc)) != IGAFD_OK || !acc) return st;
  hipLaunchKernelGGL(k_features_finish, dim3((unsigned)cdiv(c->N, kBlock)), dim3(kBlock), 0, c->stream, acc, c->feat,
                     c->N, c->p);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

template <int D, int P>
igafd_status launch_load(igafd_ctx* c, RhsDesc rhs, double* b) {
  if (D == 3 && c->modes_set) return load_across<P>(c, rhs, b);
  const Tables T = make_tables(c);
  IGAFD_HIP_CHECK(hipMemsetAsync(b, 0, sizeof(double) * c->N, c->stream));
  const int nel[3] = {c->ddir[0].nel, c->ddir[1].nel, D == 3 ? c->ddir[2].nel : 1};
  const int C3 = (D == 3) ? P + 1 : 1;
  for (int c3 = 0; c3 < C3; ++c3)
    for (int c2 = 0; c2 <= P; ++c2)
      for (int c1 = 0; c1 <= P; ++c1) {
        const int m1 = c1 < nel[0] ? (nel[0] - c1 + P) / (P + 1) : 0;
        const int m2 = c2 < nel[1] ? (nel[1] - c2 + P) / (P + 1) : 0;
        const int m3 = (D == 3) ? (c3 < nel[2] ? (nel[2] - c3 + P) / (P + 1) : 0) : 1;
        const long long blocks = (long long)m1 * m2 * m3;
        if (blocks == 0) continue;
        hipLaunchKernelGGL((k_load<D, P>), dim3((unsigned)blocks), dim3(kBlock), 0, c->stream, T, c->geom, rhs, b,
                           c1, c2, c3, m1, m2);
        IGAFD_HIP_CHECK(hipGetLastError());
      }
  return IGAFD_OK;
}

template <int D, int P>
igafd_status launch_features(igafd_ctx* c, double* acc) {
  const Tables T = make_tables(c);
  const int nel[3] = {c->ddir[0].nel, c->ddir[1].nel, D == 3 ? c->ddir[2].nel : 1};
  const int C3 = (D == 3) ? P + 1 : 1;
  for (int c3 = 0; c3 < C3; ++c3)
    for (int c2 = 0; c2 <= P; ++c2)
      for (int c1 = 0; c1 <= P; ++c1) {
        const int m1 = c1 < nel[0] ? (nel[0] - c1 + P) / (P + 1) : 0;
        const int m2 = c2 < nel[1] ? (nel[1] - c2 + P) / (P + 1) : 0;
        const int m3 = (D == 3) ? (c3 < nel[2] ? (nel[2] - c3 + P) / (P + 1) : 0) : 1;
        const long long blocks = (long long)m1 * m2 * m3;
        if (blocks == 0) continue;
        hipLaunchKernelGGL((k_features<D, P>), dim3((unsigned)blocks), dim3(kBlock), 0, c->stream, T, c->geom, acc,
                           c1, c2, c3, m1, m2);
        IGAFD_HIP_CHECK(hipGetLastError());
      }
  return IGAFD_OK;
}

template <template <int, int> class F, typename... Args>
igafd_status dispatch(int dim, int p, Args... args) {
  switch (dim * 10 + p) {
#define IGAFD_CASE(D, P) \
  case D * 10 + P:       \
    return F<D, P>::run(args...);
    IGAFD_CASE(2, 1) IGAFD_CASE(2, 2) IGAFD_CASE(2, 3) IGAFD_CASE(2, 4) IGAFD_CASE(2, 5) IGAFD_CASE(2, 6)
    IGAFD_CASE(3, 1) IGAFD_CASE(3, 2) IGAFD_CASE(3, 3) IGAFD_CASE(3, 4) IGAFD_CASE(3, 5) IGAFD_CASE(3, 6)
#undef IGAFD_CASE
    default:
      set_error("unsupported dimension/degree");
      return IGAFD_ERR_ARG;
  }
}

template <int D, int P>
struct AssembleOp {
  static igafd_status run(igafd_ctx* c, bool with_features, AsmWork* w) {
    return launch_assemble<D, P>(c, with_features, w);
  }
};
template <int D, int P>
struct FeatureOp {
  static igafd_status run(igafd_ctx* c, double* acc) { return launch_features<D, P>(c, acc); }
};
template <int D, int P>
struct LoadOp {
  static igafd_status run(igafd_ctx* c, RhsDesc f, double* b) { return launch_load<D, P>(c, f, b); }
};

}  // namespace

// Direction tables of a warped map's modes, kept by the contexts that assemble
// across the elements (A, features and load vectors read them).
igafd_status setup_modes(igafd_ctx* c) {
  c->modes_set = true;
  const int K = mode_count(c);
  if (K == 0) return IGAFD_OK;
  const int nq[3] = {c->dir[0].nel * c->dir[0].q, c->dir[1].nel * c->dir[1].q, c->dir[2].nel * c->dir[2].q};
  IGAFD_HIP_CHECK(device_malloc((void**)&c->modes, sizeof(double) * K * (2 * (size_t)nq[0] + 2 * (size_t)nq[1] + 6 * (size_t)nq[2])));
  const Modes m = modes_of(c);
  double *d0 = const_cast<double*>(m.d12[0]), *d1 = const_cast<double*>(m.d12[1]), *d3 = const_cast<double*>(m.d3);
  const dim3 grid((unsigned)cdiv((long long)(nq[0] + nq[1] + nq[2]) * K, 128));
  hipLaunchKernelGGL(k_mode_tables, grid, dim3(128), 0, c->stream, c->ddir[0].qx, c->ddir[1].qx, c->ddir[2].qx, nq[0],
                     nq[1], nq[2], c->geom, K, d0, d1, d3);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

long long load_scratch(const igafd_ctx* c) {  // 3D: the moments of one plane i3
  if (c->dim != 3 || !c->modes_set) return 0;
  const long long nq1 = (long long)c->dir[0].nel * c->dir[0].q, nq2 = (long long)c->dir[1].nel * c->dir[1].q;
  return nq1 * (nq2 + c->n[1]);
}

AsmWork::~AsmWork() {
  if (ws) block_free(ws, wait_stream(c->stream, c->device));
}

igafd_status assemble_band(igafd_ctx* c, bool with_features, AsmWork* work) {
  IGAFD_HIP_CHECK(hipMemsetAsync(c->dflag, 0, sizeof(int), c->stream));
  if (with_features) {
    const igafd_status st = block_alloc((void**)&c->feat, sizeof(float) * 8 * (size_t)c->N);
    if (st != IGAFD_OK) return st;
  }
  return dispatch<AssembleOp>(c->dim, c->p, c, with_features, work);
}

igafd_status assemble_finish(igafd_ctx* c) {
  int flag = 0;
  IGAFD_HIP_CHECK(hipMemcpyAsync(&flag, c->dflag, sizeof(int), hipMemcpyDeviceToHost, c->stream));
  IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
  if (flag) {
    set_error("det J <= 0 at a quadrature point");
    return IGAFD_ERR_GEOMETRY;
  }
  return IGAFD_OK;
}

igafd_status assemble_load(igafd_ctx* c, int rhs_kind, const double* params, int nparams, double* b) {
  if (rhs_kind < IGAFD_RHS_SINPROD || rhs_kind > IGAFD_RHS_ONE) {
    set_error("unknown right-hand side kind");
    return IGAFD_ERR_ARG;
  }
  RhsDesc f{};
  f.kind = rhs_kind;
  f.amp = rhs_kind == IGAFD_RHS_SINPROD ? c->dim * M_PI * M_PI : 1.0;
  for (int l = 0; l < 3; ++l) f.k[l] = 1.0;
  const int want = rhs_kind == IGAFD_RHS_SINPROD ? 1 + c->dim : 1;
  if (nparams != 0) {  // NULL / 0 keeps the defaults
    if (!params || nparams != want) {
      set_error("right-hand side parameters: expected " + std::to_string(want) + " values");
      return IGAFD_ERR_ARG;
    }
    f.amp = params[0];
    for (int l = 1; l < nparams; ++l) f.k[l - 1] = params[l];
  }
  return dispatch<LoadOp>(c->dim, c->p, c, f, b);
}

igafd_status spectral_bounds(igafd_ctx* c, double* qmin, double* qmax, double* qloc) {
  if (!c->bounds_valid) {
    const int nq0 = c->dir[0].nel * c->dir[0].q, nq1 = c->dir[1].nel * c->dir[1].q;
    const int nq2 = c->dim == 3 ? c->dir[2].nel * c->dir[2].q : 1;
    // partial buffer: 2 * npartial doubles = blocks (min, max, ratio) triples + the result
    int blocks = (2 * c->npartial - 3) / 3;
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) {
      set_error("internal: partial-sum buffer too small for the spectral bounds");
      return IGAFD_ERR_ARG;
    }
    double* out = c->partial + 3 * blocks;
    if (c->dim == 3)
      hipLaunchKernelGGL(k_qbounds<3>, dim3(blocks), dim3(kBlock), 0, c->stream, c->ddir[0].qx, c->ddir[1].qx,
                         c->ddir[2].qx, c->geom, nq0, nq1, nq2, c->partial);
    else
      hipLaunchKernelGGL(k_qbounds<2>, dim3(blocks), dim3(kBlock), 0, c->stream, c->ddir[0].qx, c->ddir[1].qx,
                         c->ddir[1].qx, c->geom, nq0, nq1, 1, c->partial);
    IGAFD_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_minmax, dim3(1), dim3(64), 0, c->stream, c->partial, blocks, out);
    IGAFD_HIP_CHECK(hipGetLastError());
    double h[3];
    IGAFD_HIP_CHECK(hipMemcpyAsync(h, out, sizeof(h), hipMemcpyDeviceToHost, c->stream));
    IGAFD_HIP_CHECK(hipStreamSynchronize(c->stream));
    c->qmin = h[0];
    c->qmax = h[1];
    c->qloc = h[2];
    c->bounds_valid = true;
  }
  if (qmin) *qmin = c->qmin;
  if (qmax) *qmax = c->qmax;
  if (qloc) *qloc = c->qloc;
  return IGAFD_OK;
}

igafd_status diagonals(igafd_ctx* c, double* dA, double* dP) {
  const unsigned blocks = (unsigned)((c->N + kBlock - 1) / kBlock);
  if (dA) {  // plane 0 of the band is the diagonal
    hipLaunchKernelGGL(k_copy_plane, dim3(blocks), dim3(kBlock), 0, c->stream, c->band + c->halo, dA, c->N);
    IGAFD_HIP_CHECK(hipGetLastError());
  }
  if (dP) {
    const DevDir* d = c->ddir;
    hipLaunchKernelGGL(k_diagP, dim3(blocks), dim3(kBlock), 0, c->stream, d[0].diagM, d[0].diagK, d[1].diagM,
                       d[1].diagK, d[2].diagM, d[2].diagK, c->n[0], c->n[1], c->N, c->dim, dP);
    IGAFD_HIP_CHECK(hipGetLastError());
  }
  return IGAFD_OK;
}

igafd_status features(igafd_ctx* c, float* feat) {
  if (c->feat) {  // assembled with A at setup
    IGAFD_HIP_CHECK(
        hipMemcpyAsync(feat, c->feat, sizeof(float) * 8 * (size_t)c->N, hipMemcpyDeviceToDevice, c->stream));
    return IGAFD_OK;
  }
  double* acc = nullptr;
  IGAFD_HIP_CHECK(device_malloc((void**)&acc, sizeof(double) * 8 * (size_t)c->N));
  igafd_status st = features_into(c, acc, feat);
  (void)hipStreamSynchronize(c->stream);
  (void)hipFree(acc);
  return st;
}

igafd_status features_into(igafd_ctx* c, double* acc, float* feat) {
  const unsigned blocks = (unsigned)((c->N + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_zero, dim3((unsigned)((8 * c->N + kBlock - 1) / kBlock)), dim3(kBlock), 0, c->stream, acc,
                     8 * c->N);
  IGAFD_HIP_CHECK(hipGetLastError());
  igafd_status st = dispatch<FeatureOp>(c->dim, c->p, c, acc);
  if (st != IGAFD_OK) return st;
  hipLaunchKernelGGL(k_features_finish, dim3(blocks), dim3(kBlock), 0, c->stream, acc, feat, c->N, c->p);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

// t_i = 1/2 log(P_ii / A_ii) (log = 1) or S_i = sqrt(P_ii / A_ii) (log = 0),
// diag(P) from the univariate diagonals (Sec. 3 Kronecker sum)
__global__ void k_diag_ratio(const double* __restrict__ band0, const double* m1, const double* k1, const double* m2,
                             const double* k2, const double* m3, const double* k3, int n1, int n2, long long N,
                             int dim, int log_form, float* __restrict__ t, double* __restrict__ S) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const double dP = diagP_at(m1, k1, m2, k2, m3, k3, n1, n2, dim, i);
  if (log_form)
    t[i] = (float)(0.5 * log(dP / band0[i]));
  else
    S[i] = sqrt(dP / band0[i]);
}

igafd_status scaling_targets(igafd_ctx* c, float* t) {
  const unsigned blocks = (unsigned)((c->N + kBlock - 1) / kBlock);
  const DevDir* d = c->ddir;
  hipLaunchKernelGGL(k_diag_ratio, dim3(blocks), dim3(kBlock), 0, c->stream, c->band + c->halo, d[0].diagM,
                     d[0].diagK, d[1].diagM, d[1].diagK, d[2].diagM, d[2].diagK, c->n[0], c->n[1], c->N, c->dim, 1, t,
                     nullptr);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status diag_ratio_scaling(igafd_ctx* c, double* S) {
  const unsigned blocks = (unsigned)((c->N + kBlock - 1) / kBlock);
  const DevDir* d = c->ddir;
  hipLaunchKernelGGL(k_diag_ratio, dim3(blocks), dim3(kBlock), 0, c->stream, c->band + c->halo, d[0].diagM,
                     d[0].diagK, d[1].diagM, d[1].diagK, d[2].diagM, d[2].diagK, c->n[0], c->n[1], c->N, c->dim, 0,
                     nullptr, S);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

}  // namespace igafd
