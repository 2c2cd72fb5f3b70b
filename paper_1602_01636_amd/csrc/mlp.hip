// Learned diagonal scaling S = exp(MLP(features)) for the preconditioner
// S P^-1 S.  The paper observes that P degrades when Q varies strongly
// (Sec. 3, after Prop. 1) and leaves improving it to future work; this network
// predicts, from per-dof averages of |det J| J^-1 J^-T, kappa and p, the log of
// the diagonal ratio t = 1/2 log(P_ii / A_ii), trained on pairs generated by
// the solver's own assembly.
//
// Network: 8 -> 64 -> 64 -> 1, tanh hidden layers, BF16 weights, FP32
// accumulation (MFMA v_mfma_f32_16x16x16_bf16), FP32 master weights and Adam.
//
// Layout trick: one wave handles 16 samples and computes every layer
// transposed, D^T = W X^T.  The MFMA result holds sample (lane % 16) and
// neurons 4 (lane / 16) + r, which is exactly the B-operand layout of the next
// layer's contraction over neurons, so activations never leave registers in
// the forward pass or in the back-propagation of the input gradient.  Weight
// gradients contract over samples: each wave transposes its 16-sample tiles
// through LDS, accumulates them in MFMA registers over all its sample groups,
// and the waves of a block add to one partial in LDS; a fixed-order reduction
// over the blocks finishes them, with the Adam step (deterministic, no atomics).
#include <cmath>
#include <cstring>
#include <random>

#include "internal.h"

struct igafd_mlp {
  hipStream_t stream = nullptr;
  float* theta = nullptr;    // FP32 master parameters (layout: igafd::MlpLayout)
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  float* grad = nullptr;
  float* partial = nullptr;  // per-block partial gradients (+ loss)
  float* norm = nullptr;     // mean[8], 1/std[8]
  short* w1b = nullptr;      // BF16 W1 as [64][16] (inputs zero padded)
  short* w2b = nullptr;      // BF16 W2 as [64][64]
  short* w2tb = nullptr;     // BF16 W2^T
  float* loss_dev = nullptr;
  int step = 0;
};

namespace igafd {
namespace {

constexpr int NIN = 8, NH = 64;
constexpr int OW1 = 0, OB1 = OW1 + NH * NIN, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH, OB3 = OW3 + NH;
constexpr int NPARAM = OB3 + 1;  // 4801
constexpr int MAXWAVES = 1024;
// waves per block: two when training, so that the 512 waves of an 8192-sample
// batch reach every CU and a block's sums take one step in LDS
constexpr int wpb(int train) { return train ? 2 : kBlock / 64; }

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));

__device__ inline short bf16_of(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (short)(u >> 16);
}
__device__ inline float float_of(short h) { return __uint_as_float(((unsigned)(unsigned short)h) << 16); }

__device__ inline f4_t mma(s4_t a, s4_t b, f4_t c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }

__device__ inline s4_t load4(const short* p) { return *reinterpret_cast<const s4_t*>(p); }

__device__ inline float sum_over_samples(float v) {  // over the 16 lanes of one lane group
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 4, 64);
  v += __shfl_xor(v, 8, 64);
  return v;
}

// TRAIN = 0: t (and S = exp t) for n samples.  TRAIN = 1: gradients of
// L = (1/n) sum (t - target)^2 into per-block partials.
template <int TRAIN>
__global__ __launch_bounds__(64 * wpb(TRAIN)) void k_mlp(const float* __restrict__ theta, const short* __restrict__ w1b,
                                                const short* __restrict__ w2b, const short* __restrict__ w2tb,
                                                const float* __restrict__ norm, const float* __restrict__ feat,
                                                const float* __restrict__ target, long long n, float* __restrict__ t_out,
                                                double* __restrict__ S_out, float* __restrict__ partial) {
  constexpr int WPB = wpb(TRAIN);
  __shared__ short s_dz2[WPB][NH][16];
  __shared__ short s_h1[WPB][NH][16];
  __shared__ short s_dz1[WPB][NH][16];
  __shared__ short s_f[WPB][16][16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, grp = lane >> 4;
  const int gwave = blockIdx.x * WPB + wv;
  const int nwaves = gridDim.x * WPB;
  const long long ngroups = (n + 15) / 16;

  f4_t gW2[4][4], gW1[4];
  float gb1[4][4], gb2[4][4], gw3[4][4], gb3 = 0.f, loss = 0.f;
  if (TRAIN) {
    for (int a = 0; a < 4; ++a) {
      gW1[a] = f4_t{0, 0, 0, 0};
      for (int b = 0; b < 4; ++b) gW2[a][b] = f4_t{0, 0, 0, 0};
      for (int r = 0; r < 4; ++r) gb1[a][r] = gb2[a][r] = gw3[a][r] = 0.f;
    }
  }

  // the lane's weights and biases, all loads issued before the first is waited
  // for (they were written by the previous step's kernel: every one misses L2)
  s4_t a1[4], a2[4][4], a3[4][4];
  float c1[4][4], c2[4][4], c3[4][4];
  const float c4 = theta[OB3];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    a1[m] = load4(w1b + (16 * m + col) * 16 + 4 * grp);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a2[m][k] = load4(w2b + (16 * m + col) * NH + 16 * k + 4 * grp);
      if (TRAIN) a3[m][k] = load4(w2tb + (16 * m + col) * NH + 16 * k + 4 * grp);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      c1[m][r] = theta[OB1 + 16 * m + 4 * grp + r];
      c2[m][r] = theta[OB2 + 16 * m + 4 * grp + r];
      c3[m][r] = theta[OW3 + 16 * m + 4 * grp + r];
    }
  }
  for (long long g = gwave; g < ngroups; g += nwaves) {
    const long long s = g * 16 + col;
    const bool live = s < n;
    // features of sample s, inputs 4 grp + j (zero beyond the 8 inputs)
    float fin[4];
    for (int j = 0; j < 4; ++j) {
      const int k = 4 * grp + j;
      fin[j] = (live && k < NIN) ? (feat[s * NIN + k] - norm[k]) * norm[NIN + k] : 0.f;
    }
    const s4_t bF = {bf16_of(fin[0]), bf16_of(fin[1]), bf16_of(fin[2]), bf16_of(fin[3])};
    // layer 1: z1^T = W1 f^T
    float h1[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f4_t d = mma(a1[m], bF, f4_t{0, 0, 0, 0});
#pragma unroll
      for (int r = 0; r < 4; ++r) h1[m][r] = tanhf(d[r] + c1[m][r]);
    }
    s4_t bH1[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) bH1[m] = s4_t{bf16_of(h1[m][0]), bf16_of(h1[m][1]), bf16_of(h1[m][2]), bf16_of(h1[m][3])};
    // layer 2: z2^T = W2 h1^T
    float h2[4][4];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      f4_t d = {0, 0, 0, 0};
#pragma unroll
      for (int m = 0; m < 4; ++m) d = mma(a2[o][m], bH1[m], d);
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[o][r] = tanhf(d[r] + c2[o][r]);
    }
    // layer 3: t = w3 . h2 + b3 (lane-local partial, then over the 4 lane groups)
    float part = 0.f;
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) part += c3[o][r] * h2[o][r];
    part += __shfl_xor(part, 16, 64);
    part += __shfl_xor(part, 32, 64);
    const float t = part + c4;
    if (!TRAIN) {
      if (grp == 0 && live) {
        if (t_out) t_out[s] = t;
        if (S_out) S_out[s] = exp((double)t);
      }
      continue;
    }
    const float e = live ? t - target[s] : 0.f;
    const float dt = 2.f * e / (float)n;
    if (grp == 0) {
      loss += e * e;
      gb3 += dt;
    }
    // back-propagation: dz2 = dt w3 (1 - h2^2)
    float dz2[4][4];
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dz2[o][r] = dt * c3[o][r] * (1.f - h2[o][r] * h2[o][r]);
        gw3[o][r] += dt * h2[o][r];
        gb2[o][r] += dz2[o][r];
      }
    s4_t bDz2[4];
#pragma unroll
    for (int o = 0; o < 4; ++o)
      bDz2[o] = s4_t{bf16_of(dz2[o][0]), bf16_of(dz2[o][1]), bf16_of(dz2[o][2]), bf16_of(dz2[o][3])};
    // dh1^T = W2^T dz2^T, dz1 = dh1 (1 - h1^2)
    float dz1[4][4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      f4_t d = {0, 0, 0, 0};
#pragma unroll
      for (int o = 0; o < 4; ++o) d = mma(a3[m][o], bDz2[o], d);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dz1[m][r] = d[r] * (1.f - h1[m][r] * h1[m][r]);
        gb1[m][r] += dz1[m][r];
      }
    }
    // weight gradients: transpose the tiles through LDS ([neuron][sample])
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int nrn = 16 * m + 4 * grp + r;
        s_dz2[wv][nrn][col] = bf16_of(dz2[m][r]);
        s_h1[wv][nrn][col] = bf16_of(h1[m][r]);
        s_dz1[wv][nrn][col] = bf16_of(dz1[m][r]);
      }
#pragma unroll
    for (int j = 0; j < 4; ++j) s_f[wv][4 * grp + j][col] = bF[j];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // dW2[o][i] += sum_s dz2[o][s] h1[i][s];  dW1[o][k] += sum_s dz1[o][s] f[k][s]
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const s4_t aDz2 = load4(&s_dz2[wv][16 * a + col][4 * grp]);
      const s4_t aDz1 = load4(&s_dz1[wv][16 * a + col][4 * grp]);
#pragma unroll
      for (int b = 0; b < 4; ++b) gW2[a][b] = mma(aDz2, load4(&s_h1[wv][16 * b + col][4 * grp]), gW2[a][b]);
      gW1[a] = mma(aDz1, load4(&s_f[wv][col][4 * grp]), gW1[a]);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
  if (!TRAIN) return;
  // the block's sums: an LDS image per wave, added on the way out, so that a
  // block and not a wave writes the 4802 values that k_mlp_step reads again
  __shared__ float s_sum[TRAIN ? WPB : 1][TRAIN ? NPARAM + 1 : 1];
  float* im = s_sum[wv];
  // result lane layout: row 4 grp + r, column col of each 16 x 16 tile
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int o = 16 * a + 4 * grp + r;
#pragma unroll
      for (int b = 0; b < 4; ++b) im[OW2 + o * NH + 16 * b + col] = gW2[a][b][r];
      if (col < NIN) im[OW1 + o * NIN + col] = gW1[a][r];
    }
  // per-neuron sums over the 16 sample lanes of each lane group
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v1 = sum_over_samples(gb1[m][r]);
      const float v2 = sum_over_samples(gb2[m][r]);
      const float v3 = sum_over_samples(gw3[m][r]);
      if (col == 0) {
        const int nrn = 16 * m + 4 * grp + r;
        im[OB1 + nrn] = v1;
        im[OB2 + nrn] = v2;
        im[OW3 + nrn] = v3;
      }
    }
  const float tb3 = sum_over_samples(gb3);
  const float tl = sum_over_samples(loss);
  if (lane == 0) {
    im[OB3] = tb3;
    im[NPARAM] = tl;
  }
  __syncthreads();
  static_assert(!TRAIN || WPB == 2, "a block's sum is that of two waves' images");
  float* out = partial + (long long)blockIdx.x * (NPARAM + 1);
  for (int k = threadIdx.x; k <= NPARAM; k += 64 * WPB) out[k] = s_sum[0][k] + s_sum[TRAIN ? WPB - 1 : 0][k];
}

// The parameter's BF16 copies (W1 padded to 16 inputs, W2 and W2^T).
__device__ inline void refresh_param(int k, float v, short* __restrict__ w1b, short* __restrict__ w2b,
                                     short* __restrict__ w2tb) {
  if (k < OB1) {
    w1b[(k / NIN) * 16 + k % NIN] = bf16_of(v);
  } else if (k >= OW2 && k < OB2) {
    const int q = k - OW2, o = q / NH, i = q % NH;
    w2b[q] = bf16_of(v);
    w2tb[i * NH + o] = bf16_of(v);
  }
}

// grad[k] = sum of the blocks' partials (fixed order); loss = sum / n.  With
// lr > 0 also the Adam step and the BF16 copies of the new parameter.  A block
// owns kStepCols parameters and its kStepRows rows of threads each a share of
// the partials, eight loads in flight, so the 256 partials of an 8192-sample
// batch take two trips to memory and not 256 in sequence: 4.0 us, where
// reduction, Adam and copies in three launches, one thread per parameter over
// the partials of 512 waves, took 113.6 + 4.7 + 4.6 us.  The step is bound by
// the dependent chain of k_mlp's one sample group per wave (16.7 us; 20.1 with
// the weights loaded where they are used and four waves on half of the CUs).
constexpr int kStepCols = 32, kStepRows = 16;
__global__ __launch_bounds__(kStepCols * kStepRows) void k_mlp_step(const float* __restrict__ partial, int nb,
                                                                    float* __restrict__ grad,
                                                                    float* __restrict__ loss, long long n, float lr,
                                                                    float c1, float c2, float* __restrict__ theta,
                                                                    float* __restrict__ m, float* __restrict__ v,
                                                                    short* __restrict__ w1b, short* __restrict__ w2b,
                                                                    short* __restrict__ w2tb) {
  __shared__ float s[kStepRows][kStepCols + 1];
  const int c = threadIdx.x % kStepCols, row = threadIdx.x / kStepCols;
  const int k = blockIdx.x * kStepCols + c;
  float a = 0.f;
  if (k <= NPARAM) {
#pragma unroll 8
    for (int w = row; w < nb; w += kStepRows) a += partial[(long long)w * (NPARAM + 1) + k];
  }
  s[row][c] = a;
  __syncthreads();
  if (row != 0 || k > NPARAM) return;
  float g = 0.f;
#pragma unroll
  for (int r = 0; r < kStepRows; ++r) g += s[r][c];
  if (k == NPARAM) {
    *loss = g / (float)n;
    return;
  }
  grad[k] = g;
  if (!(lr > 0.f)) return;
  const float b1 = 0.9f, b2 = 0.999f;
  const float mk = b1 * m[k] + (1.f - b1) * g, vk = b2 * v[k] + (1.f - b2) * g * g;
  m[k] = mk;
  v[k] = vk;
  const float t = theta[k] - lr * (mk / c1) / (sqrtf(vk / c2) + 1e-8f);
  theta[k] = t;
  refresh_param(k, t, w1b, w2b, w2tb);
}

// BF16 copies of all weight matrices; the padding inputs of W1 zero
__global__ void k_mlp_refresh(const float* __restrict__ theta, short* __restrict__ w1b, short* __restrict__ w2b,
                              short* __restrict__ w2tb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < NPARAM) refresh_param(k, theta[k], w1b, w2b, w2tb);
  if (k < NH * (16 - NIN)) w1b[(k / (16 - NIN)) * 16 + NIN + k % (16 - NIN)] = 0;
}

// mean and 1/std of each of the 8 inputs (one block per input, fixed order)
__global__ void k_mlp_norm(const float* __restrict__ feat, long long n, float* __restrict__ norm) {
  __shared__ double red[2][kBlock];
  const int ch = blockIdx.x;
  double s = 0.0, s2 = 0.0;
  for (long long i = threadIdx.x; i < n; i += kBlock) {
    const double f = feat[i * NIN + ch];
    s += f;
    s2 += f * f;
  }
  red[0][threadIdx.x] = s;
  red[1][threadIdx.x] = s2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int k = 0; k < kBlock; ++k) {
      a += red[0][k];
      b += red[1][k];
    }
    const double mean = a / (double)n;
    const double var = b / (double)n - mean * mean;
    norm[ch] = (float)mean;
    norm[NIN + ch] = var > 1e-20 ? (float)(1.0 / sqrt(var)) : 1.f;
  }
}

int blocks_for(long long n, int train) {
  const long long groups = (n + 15) / 16, w = groups < MAXWAVES ? groups : MAXWAVES;
  return (int)((w + wpb(train) - 1) / wpb(train));
}

igafd_status refresh(igafd_mlp* M) {
  hipLaunchKernelGGL(k_mlp_refresh, dim3((NPARAM + 255) / 256), dim3(256), 0, M->stream, M->theta, M->w1b, M->w2b,
                     M->w2tb);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

// gradient and loss; with lr > 0 also the Adam step number `step`
igafd_status gradient(igafd_mlp* M, const float* feat, const float* target, long long n, float lr, int step) {
  const int nb = blocks_for(n, 1);
  hipLaunchKernelGGL((k_mlp<1>), dim3(nb), dim3(64 * wpb(1)), 0, M->stream, M->theta, M->w1b, M->w2b, M->w2tb, M->norm,
                     feat, target, n, nullptr, nullptr, M->partial);
  IGAFD_HIP_CHECK(hipGetLastError());
  const float c1 = 1.f - std::pow(0.9f, (float)step), c2 = 1.f - std::pow(0.999f, (float)step);
  hipLaunchKernelGGL(k_mlp_step, dim3((NPARAM + kStepCols) / kStepCols), dim3(kStepCols * kStepRows), 0, M->stream,
                     M->partial, nb, M->grad, M->loss_dev, n, lr, c1, c2, M->theta, M->adam_m, M->adam_v, M->w1b,
                     M->w2b, M->w2tb);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

}  // namespace
}  // namespace igafd

using namespace igafd;

extern "C" {

igafd_status igafd_mlp_create(unsigned long long seed, void* stream, igafd_mlp** out) {
  if (!out) {
    set_error("null argument");
    return IGAFD_ERR_ARG;
  }
  igafd_mlp* M = new igafd_mlp();
  M->stream = (hipStream_t)stream;
  *out = nullptr;
  const size_t pb = sizeof(float) * NPARAM;
#define IGAFD_M(ptr, bytes)                                         \
  if (device_malloc((void**)&(ptr), (bytes)) != hipSuccess) {           \
    igafd_mlp_destroy(M);                                           \
    set_error("allocation of the network buffers failed");          \
    return IGAFD_ERR_ALLOC;                                         \
  }
  IGAFD_M(M->theta, pb) IGAFD_M(M->adam_m, pb) IGAFD_M(M->adam_v, pb) IGAFD_M(M->grad, pb)
  IGAFD_M(M->partial, sizeof(float) * (size_t)(MAXWAVES / wpb(1)) * (NPARAM + 1)) IGAFD_M(M->norm, sizeof(float) * 2 * NIN)
  IGAFD_M(M->w1b, sizeof(short) * NH * 16) IGAFD_M(M->w2b, sizeof(short) * NH * NH)
  IGAFD_M(M->w2tb, sizeof(short) * NH * NH) IGAFD_M(M->loss_dev, sizeof(float))
#undef IGAFD_M
  // Glorot-uniform weights from a seeded generator, zero biases, identity normalisation
  std::vector<float> th(NPARAM, 0.f), nm(2 * NIN, 0.f);
  std::mt19937_64 gen(seed);
  auto fill = [&](int off, int fan_in, int fan_out, int count) {
    const float a = std::sqrt(6.f / (fan_in + fan_out));
    std::uniform_real_distribution<float> U(-a, a);
    for (int k = 0; k < count; ++k) th[off + k] = U(gen);
  };
  fill(OW1, NIN, NH, NH * NIN);
  fill(OW2, NH, NH, NH * NH);
  fill(OW3, NH, 1, NH);
  for (int k = 0; k < NIN; ++k) nm[NIN + k] = 1.f;
  std::vector<float> zeros(NPARAM, 0.f);
  if (hipMemcpy(M->theta, th.data(), sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(M->adam_m, zeros.data(), sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(M->adam_v, zeros.data(), sizeof(float) * NPARAM, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(M->norm, nm.data(), sizeof(float) * 2 * NIN, hipMemcpyHostToDevice) != hipSuccess ||
      refresh(M) != IGAFD_OK || hipStreamSynchronize(M->stream) != hipSuccess) {
    igafd_mlp_destroy(M);
    set_error("network initialisation failed");
    return IGAFD_ERR_HIP;
  }
  *out = M;
  return IGAFD_OK;
}

void igafd_mlp_destroy(igafd_mlp* M) {
  if (!M) return;
  if (M->stream) (void)hipStreamSynchronize(M->stream);
  for (void* p : {(void*)M->theta, (void*)M->adam_m, (void*)M->adam_v, (void*)M->grad, (void*)M->partial,
                  (void*)M->norm, (void*)M->w1b, (void*)M->w2b, (void*)M->w2tb, (void*)M->loss_dev})
    if (p) (void)hipFree(p);
  delete M;
}

igafd_status igafd_mlp_fit_normalization(igafd_mlp* M, const float* feat, long long n) {
  if (!M || !feat || n < 1) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  hipLaunchKernelGGL(k_mlp_norm, dim3(NIN), dim3(kBlock), 0, M->stream, feat, n, M->norm);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status igafd_mlp_get_params(const igafd_mlp* M, float* host) {
  if (!M || !host) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  IGAFD_HIP_CHECK(hipStreamSynchronize(M->stream));
  IGAFD_HIP_CHECK(hipMemcpy(host, M->theta, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
  IGAFD_HIP_CHECK(hipMemcpy(host + NPARAM, M->norm, sizeof(float) * 2 * NIN, hipMemcpyDeviceToHost));
  return IGAFD_OK;
}

igafd_status igafd_mlp_set_params(igafd_mlp* M, const float* host) {
  if (!M || !host) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  IGAFD_HIP_CHECK(hipStreamSynchronize(M->stream));
  IGAFD_HIP_CHECK(hipMemcpy(M->theta, host, sizeof(float) * NPARAM, hipMemcpyHostToDevice));
  IGAFD_HIP_CHECK(hipMemcpy(M->norm, host + NPARAM, sizeof(float) * 2 * NIN, hipMemcpyHostToDevice));
  return refresh(M);
}

igafd_status igafd_mlp_forward(igafd_mlp* M, const float* feat, long long n, float* t_out, double* S_out) {
  if (!M || !feat || n < 0) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  if (n == 0) return IGAFD_OK;
  hipLaunchKernelGGL((k_mlp<0>), dim3(blocks_for(n, 0)), dim3(64 * wpb(0)), 0, M->stream, M->theta, M->w1b, M->w2b, M->w2tb,
                     M->norm, feat, nullptr, n, t_out, S_out, nullptr);
  IGAFD_HIP_CHECK(hipGetLastError());
  return IGAFD_OK;
}

igafd_status igafd_mlp_gradient(igafd_mlp* M, const float* feat, const float* target, long long n, float* grad_host,
                                float* loss_host) {
  if (!M || !feat || !target || n < 1) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  igafd_status s = gradient(M, feat, target, n, 0.f, 1);
  if (s != IGAFD_OK) return s;
  IGAFD_HIP_CHECK(hipStreamSynchronize(M->stream));
  if (grad_host) IGAFD_HIP_CHECK(hipMemcpy(grad_host, M->grad, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
  if (loss_host) IGAFD_HIP_CHECK(hipMemcpy(loss_host, M->loss_dev, sizeof(float), hipMemcpyDeviceToHost));
  return IGAFD_OK;
}

igafd_status igafd_mlp_train_step(igafd_mlp* M, const float* feat, const float* target, long long n, float lr,
                                  float* loss_host) {
  if (!M || !feat || !target || n < 1 || !(lr > 0.f)) {
    set_error("bad arguments");
    return IGAFD_ERR_ARG;
  }
  igafd_status s = gradient(M, feat, target, n, lr, M->step + 1);
  if (s != IGAFD_OK) return s;
  M->step += 1;
  if (loss_host) {
    IGAFD_HIP_CHECK(hipMemcpyAsync(loss_host, M->loss_dev, sizeof(float), hipMemcpyDeviceToHost, M->stream));
    IGAFD_HIP_CHECK(hipStreamSynchronize(M->stream));
  }
  return IGAFD_OK;
}

int igafd_mlp_num_params(void) { return NPARAM; }

}  // extern "C"
