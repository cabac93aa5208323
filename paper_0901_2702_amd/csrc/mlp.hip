// Learned initialiser on gfx950: a multilayer perceptron (K0 -> 256 -> 256 ->
// 256 -> 32 (10 used), GELU with the erf normal CDF) evaluated and trained with bfloat16 MFMA
// (v_mfma_f32_16x16x32_bf16, float32 accumulation) and Adam on float32
// master weights.
//
// The paper initialises B, gamma and v_los with small back-propagation
// networks trained on synthetic filtered noisy profiles, with early stopping
// on a control set (Sect. 5).  Here one network proposes all ten starting
// parameters, trained on profiles synthesised by the library's own forward
// model.
//
// Every product is C = A . Bt^T with A [M][Kd] and Bt [N][Kd] both contiguous
// along Kd, so each lane fetches its 8-element MFMA fragments with one
// 16-byte load:  forward  X [B][K] . Wt [N][K]^T;  input gradient
// dZ [B][N] . W [K][N]^T;  weight gradient X^T [K][B] . dZ^T [N][B]^T (in the
// [in][out] order of the master weights, so that the Adam kernel reads it
// coalesced), split along the batch into MLP_SPLITK partial sums that the
// Adam kernel adds.
//
// A training step is three launches.  Everything that concerns one row of the
// batch (inputs, four layers, loss, the gradient down to the first layer's
// pre-activation) runs in one workgroup per few rows, which leaves only the
// transposed activations and gradients behind (train_rows_kernel); all weight
// and bias gradients follow in one launch, and Adam.  One launch per product
// and element-wise pass, 15 per step, spent 99 us of a step of 4,096 rows in
// kernels of 3 to 10 us that mostly waited for their first loads.
#include <hip/hip_runtime.h>

#include "me_device.h"
#include "mlp.h"

namespace vfisv {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// GELU(z) = z Phi(z) with the exact (erf) normal CDF Phi, evaluated
// branch-free from erfc(|z| / sqrt 2) by the rational-exponential
// approximation of Abramowitz & Stegun 7.1.26 (Hastings):
//   erfc(x) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-x^2),
//   t = 1 / (1 + p x),
// absolute error below 1.5e-7 -- under a thousandth of the bfloat16 step the
// activations are rounded to.  Phi(z) = 1 - erfc(x) / 2 for z >= 0 and
// erfc(x) / 2 for z < 0 (so the negative tail keeps its relative accuracy);
// the halves are folded into the coefficients.  The device library's erff
// branches on |x| (divergent lanes, two polynomials) and took twice the
// instructions of the network's epilogues.
struct PhiPdf {
  float Phi;  // Phi(z)
  float e;    // exp(-z^2 / 2)
};
__device__ __forceinline__ PhiPdf phi_pdf(float z) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = frcp(fmaf(0.3275911f, x, 1.f));
  float p = fmaf(t, 0.5f * 1.061405429f, 0.5f * -1.453152027f);
  p = fmaf(t, p, 0.5f * 1.421413741f);
  p = fmaf(t, p, 0.5f * -0.284496736f);
  p = fmaf(t, p, 0.5f * 0.254829592f);
  // exp(-z^2 / 2) = 2^(-z^2 log2(e) / 2)
  const float e = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);
  const float h = t * p * e;  // erfc(x) / 2
  return PhiPdf{z >= 0.f ? 1.f - h : h, e};
}
__device__ __forceinline__ float gelu(float z) { return z * phi_pdf(z).Phi; }
// d/dz [z Phi(z)] = Phi(z) + z phi(z), phi(z) = exp(-z^2 / 2) / sqrt(2 pi)
__device__ __forceinline__ float gelu_grad(float z) {
  const PhiPdf f = phi_pdf(z);
  return fmaf(z * 0.39894228040143268f, f.e, f.Phi);
}

// ---- training: rows ----------------------------------------------------------
// MFMA 16x16x32 lane layout: lane l feeds A row (l & 15) and B column (l & 15)
// with k = 8 (l >> 4) .. +7, and receives C rows 4 (l >> 4) .. +3 of column
// (l & 15).  Each element is one chain of MFMAs over ascending k.
// Transposed copies store four consecutive rows with one 8-byte write.
__device__ __forceinline__ void store4_bf16(bf16* p, float v0, float v1, float v2, float v3) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
  bf16x4 v;
  v[0] = (bf16)v0;
  v[1] = (bf16)v1;
  v[2] = (bf16)v2;
  v[3] = (bf16)v3;
  *(bf16x4*)p = v;
}

constexpr int LDH = MLP_H + 8;  // row of 256 activations in LDS
constexpr int TW = 8;           // waves of a workgroup; wave w owns columns [32 w, 32 w + 32)
constexpr int TCB = MLP_H / (16 * TW);
constexpr int LDZ = MLP_OUT + 8;

struct TrainRowsArgs {
  const float* stokes;
  const int32_t* rows;  // batch row -> sample (nullptr: the same)
  const float* targets;
  int64_t M, cap;
  int n_in, K0;
  const float* mean;
  const float* istd;
  const bf16* Wt[4];
  const bf16* Wk[4];
  const float* bias[4];
  bf16* X0t;
  bf16* Yt[3];
  bf16* dZt[4];
  double* loss;
};

// This wave's fragments of NK k-steps of a weight matrix (rows of ld).
template <int NK>
struct TrainW {
  bf16x8 f[NK][TCB];
  __device__ __forceinline__ void fetch(const bf16* W, int ld, int wave, int l) {
    const bf16* p = W + (int64_t)(wave * 16 * TCB + (l & 15)) * ld + (l >> 4) * 8;
#pragma unroll
    for (int s = 0; s < NK; ++s)
#pragma unroll
      for (int cb = 0; cb < TCB; ++cb) f[s][cb] = *(const bf16x8*)(p + (int64_t)cb * 16 * ld + 32 * s);
  }
};

template <int RB, int NK>
__device__ __forceinline__ void train_product(const bf16* in, int ldin, const TrainW<NK>& w,
                                              f32x4 (&acc)[RB][TCB], int l) {
#pragma unroll
  for (int s = 0; s < NK; ++s) {
    bf16x8 a[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      a[rb] = *(const bf16x8*)(in + (rb * 16 + (l & 15)) * ldin + 32 * s + (l >> 4) * 8);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < TCB; ++cb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], w.f[s][cb], acc[rb][cb], 0, 0, 0);
  }
}

// out[rb][cb] = f(acc, index) as bfloat16, to the tile h and transposed to t
template <int RB, class F>
__device__ __forceinline__ void train_epilogue(const f32x4 (&acc)[RB][TCB], bf16* h, bf16* t,
                                               int64_t cap, int64_t m0, int wave, int l, F f) {
#pragma unroll
  for (int cb = 0; cb < TCB; ++cb) {
    const int col = wave * 16 * TCB + cb * 16 + (l & 15);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const int row = rb * 16 + (l >> 4) * 4;
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] = f(acc[rb][cb][j], rb, cb, j);
        if (h) h[(row + j) * LDH + col] = (bf16)v[j];
      }
      store4_bf16(t + (int64_t)col * cap + m0 + row, v[0], v[1], v[2], v[3]);
    }
  }
}

constexpr int64_t TRAIN_RB2_ROWS = 131072;
template <int RB>
constexpr size_t train_lds_bytes(int K0) {
  const size_t R = 16 * RB;
  return R * (sizeof(bf16) * (K0 + 8 + 2 * LDH + LDZ) + sizeof(float) * (MLP_OUT + 1 + MLP_OUT));
}

// 16 RB rows per workgroup.  Bound by its own chain of seven dependent
// products and by the weights' way from L2 (560 KB per workgroup): a layer's
// weights are fetched two products ahead into registers, pre-activations stay
// there (in float32) for the way back.  256 workgroups for a batch of 4,096
// (RB = 1); RB = 2 halves the weights' reads, which tells only where they are
// the larger part of the traffic: 524,288 rows 4.3 ms with RB = 1, 4.05 with
// RB = 2, 65,536 equal, 16,384 138 us against 142.  (RB = 2 does not fit the
// registers: 256 bytes of scratch per lane, in those times.)
template <int RB>
__global__ __launch_bounds__(TW * 64, 2) void train_rows_kernel(const TrainRowsArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int R = 16 * RB, NT = TW * 64;
  const int ldx = a.K0 + 8;
  bf16* const xs = (bf16*)smem;   // [R][K0 + 8]
  bf16* const h0 = xs + R * ldx;  // [R][LDH]
  bf16* const h1 = h0 + R * LDH;
  bf16* const dz = h1 + R * LDH;  // [R][LDZ]
  float* const y4 = (float*)(dz + R * LDZ);  // [R][MLP_OUT + 1]
  float* const red = y4 + R * (MLP_OUT + 1); // [R * MLP_OUT]
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  // neighbouring rows on one XCD: they share the transposed outputs' lines
  const unsigned nb = gridDim.x, b = blockIdx.x;
  const int64_t m0 = (int64_t)(nb % 8 == 0 ? (b % 8) * (nb / 8) + b / 8 : b) * R;
  constexpr int NH = MLP_H / 32;
  // the first layer's weights, NF k-steps ahead (a step of 32 rows of 1,248
  // inputs 90 us with one at a time, 78 like this)
  constexpr int NF = 4;
  TrainW<1> w0[NF];
  TrainW<1>& w1 = w0[0];
  TrainW<NH> wa, wb;
  const int steps = a.K0 / 32;
  // inputs, and the targets of this thread's outputs
  for (int i = tid; i < R * a.K0; i += NT) {
    const int r = i / a.K0, k = i - r * a.K0;
    const int64_t src = a.rows ? (int64_t)a.rows[m0 + r] : m0 + r;
    const float x = k < a.n_in ? (a.stokes[src * a.n_in + k] - a.mean[k]) * a.istd[k] : 0.f;
    xs[r * ldx + k] = (bf16)x;
  }
  float target[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int e = tid + NT * i, r = e / MLP_OUT, c = e % MLP_OUT;
    const int64_t src = a.rows ? (int64_t)a.rows[m0 + r] : m0 + r;
    target[i] = c < MLP_NCODE ? a.targets[src * MLP_NCODE + c] : 0.f;
  }
  w1.fetch(a.Wt[0], a.K0, wave, l);
  if (steps > 1) {
#pragma unroll
    for (int i = 1; i < NF; ++i)
      if (i < steps) w0[i].fetch(a.Wt[0] + 32 * i, a.K0, wave, l);
  }
  float bias[3][TCB];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int cb = 0; cb < TCB; ++cb) bias[i][cb] = a.bias[i][wave * 16 * TCB + cb * 16 + (l & 15)];
  wa.fetch(a.Wt[1], MLP_H, wave, l);
  __syncthreads();
  wb.fetch(a.Wt[2], MLP_H, wave, l);
  for (int i = tid; i < a.K0 * (R / 8); i += NT) {
    const int k = i / (R / 8), g = 8 * (i % (R / 8));
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = xs[(g + j) * ldx + k];
    *(bf16x8*)(a.X0t + (int64_t)k * a.cap + m0 + g) = v;
  }
  float z[3][RB][TCB][4];
  const auto zero = [](f32x4 (&acc)[RB][TCB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < TCB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  f32x4 acc[RB][TCB];
  // first layer: xs -> h0
  zero(acc);
  if (steps == 1) {
    train_product<RB, 1>(xs, ldx, w1, acc, l);
  } else {
    for (int k = 0; k < steps; k += NF) {
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        if (k + i >= steps) break;
        train_product<RB, 1>(xs + 32 * (k + i), ldx, w0[i], acc, l);
        if (k + i + NF < steps) w0[i].fetch(a.Wt[0] + 32 * (k + i + NF), a.K0, wave, l);
      }
    }
  }
  const auto hidden = [&](int layer, bf16* h) {
    train_epilogue<RB>(acc, h, a.Yt[layer], a.cap, m0, wave, l, [&](float c, int rb, int cb, int j) {
      z[layer][rb][cb][j] = c + bias[layer][cb];
      return gelu(z[layer][rb][cb][j]);
    });
  };
  const auto back = [&](int layer, bf16* h) {
    train_epilogue<RB>(acc, h, a.dZt[layer], a.cap, m0, wave, l, [&](float c, int rb, int cb, int j) {
      return c * gelu_grad(z[layer][rb][cb][j]);
    });
  };
  hidden(0, h0);
  __syncthreads();
  // second layer: h0 -> h1
  zero(acc);
  train_product<RB, NH>(h0, LDH, wa, acc, l);
  wa.fetch(a.Wk[2], MLP_H, wave, l);
  hidden(1, h1);
  __syncthreads();
  // third layer: h1 -> h0
  zero(acc);
  train_product<RB, NH>(h1, LDH, wb, acc, l);
  // the output layer's products: waves 0 .. 2 RB - 1, a tile each
  const bool out_wave = wave < 2 * RB;
  const int out_col = (wave & 1) * 16 + (l & 15);
  bf16x8 wo[NH];
  if (out_wave) {
#pragma unroll
    for (int s = 0; s < NH; ++s)
      wo[s] = *(const bf16x8*)(a.Wt[3] + (int64_t)out_col * MLP_H + 32 * s + (l >> 4) * 8);
  }
  w1.fetch(a.Wk[3], MLP_OUT, wave, l);
  hidden(2, h0);
  __syncthreads();
  if (out_wave) {
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    const int r0 = (wave >> 1) * 16;
#pragma unroll
    for (int s = 0; s < NH; ++s)
      o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          *(const bf16x8*)(h0 + (r0 + (l & 15)) * LDH + 32 * s + (l >> 4) * 8), wo[s], o, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      y4[(r0 + (l >> 4) * 4 + j) * (MLP_OUT + 1) + out_col] = o[j] + a.bias[3][out_col];
  }
  wb.fetch(a.Wk[1], MLP_H, wave, l);
  __syncthreads();
  // loss and its gradient
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int e = tid + NT * i, r = e / MLP_OUT, c = e % MLP_OUT;
    const float d = c < MLP_NCODE ? y4[r * (MLP_OUT + 1) + c] - target[i] : 0.f;
    red[e] = d * d;
    dz[r * LDZ + c] = (bf16)(2.f * d / (float)(a.M * MLP_NCODE));
  }
  __syncthreads();
  if (wave < R / 8) {  // 8 rows' squares, halved pairwise from 128 apart down to neighbours
    const float* q = red + 256 * wave + l;
    float s = (q[0] + q[128]) + (q[64] + q[192]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_down(s, off);
    if (l == 0) atomicAdd(a.loss, (double)s);
  }
  for (int i = tid; i < MLP_OUT * (R / 8); i += NT) {
    const int c = i / (R / 8), g = 8 * (i % (R / 8));
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = dz[(g + j) * LDZ + c];
    *(bf16x8*)(a.dZt[3] + (int64_t)c * a.cap + m0 + g) = v;
  }
  // back through the output layer, dz -> h1, and the third and second, h1 -> h0 -> out
  zero(acc);
  train_product<RB, 1>(dz, LDZ, w1, acc, l);
  back(2, h1);
  __syncthreads();
  zero(acc);
  train_product<RB, NH>(h1, LDH, wa, acc, l);
  back(1, h0);
  __syncthreads();
  zero(acc);
  train_product<RB, NH>(h0, LDH, wb, acc, l);
  back(0, nullptr);
}

// ---- training: weight and bias gradients ------------------------------------
// One launch for all four layers.  Weights: dW[in][out] = X^T[in][B] .
// dZ^T[out][B]^T, a wave per 32 x 32 tile and batch chunk (2 x 2 MFMA tiles;
// the fragments of KC k-steps are loaded before the first MFMA of the group,
// so that one memory latency serves them all).  Biases: db[n] = sum of
// dZ^T[n][:], a workgroup per column; the batch dimension is contiguous, so
// each thread reads 8 values per load (M and cap are multiples of 32: 16-byte
// aligned rows), then a wave reduction and one LDS step combine the 256
// partial sums.  (A wave per column: 17.4 us instead of 15.2 for 4,096 rows.)
constexpr int GT = 2;   // 16 x 16 MFMA tiles per wave along each of in and out
constexpr int GKC = 8;  // k-steps loaded per group
constexpr int GRAD_XCDS = 8;
static_assert(MLP_SPLITK % GRAD_XCDS == 0, "chunks per XCD");
// workgroups of four tiles per XCD
__host__ __device__ constexpr int grad_blocks(int n_tiles) {
  return (n_tiles * (MLP_SPLITK / GRAD_XCDS) + 3) / 4;
}
struct GradArgs {
  const bf16* Xt[4];
  const bf16* dZt[4];
  float* part[4];  // [split][in][out]
  float* grad_b[4];
  int in_dim[4], out_dim[4];
  int first_tile[5];  // first tile of each layer (of one chunk); then the total
  int first_col[5];   // first bias column of each layer; then the total
  int64_t M, cap, chunk;
};

__device__ __forceinline__ void weight_grad_tile(const GradArgs& a, int tile, int split,
                                                 int l) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i) q = tile >= a.first_tile[i] ? i : q;
  const int t = tile - a.first_tile[q], nn = a.out_dim[q] / (16 * GT);
  const int n0 = t % nn * 16 * GT, m0 = t / nn * 16 * GT;
  const int64_t kbeg = split * a.chunk;
  const int64_t kend = kbeg + a.chunk < a.M ? kbeg + a.chunk : a.M;
  const int lr = l & 15, lk = (l >> 4) * 8;
  const bf16* arow = a.Xt[q] + (int64_t)(m0 + lr) * a.cap + lk;
  const bf16* bcol = a.dZt[q] + (int64_t)(n0 + lr) * a.cap + lk;
  f32x4 acc[GT][GT];
#pragma unroll
  for (int rb = 0; rb < GT; ++rb)
#pragma unroll
    for (int cb = 0; cb < GT; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 zero;
#pragma unroll
  for (int i = 0; i < 8; ++i) zero[i] = (bf16)0.f;
  for (int64_t k0 = kbeg; k0 < kend; k0 += 32 * GKC) {
    bf16x8 x[GKC][GT], y[GKC][GT];
#pragma unroll
    for (int kc = 0; kc < GKC; ++kc) {
      const int64_t k = k0 + 32 * kc;
#pragma unroll
      for (int i = 0; i < GT; ++i) {
        x[kc][i] = k < kend ? *(const bf16x8*)(arow + 16 * i * a.cap + k) : zero;
        y[kc][i] = k < kend ? *(const bf16x8*)(bcol + 16 * i * a.cap + k) : zero;
      }
    }
#pragma unroll
    for (int kc = 0; kc < GKC; ++kc) {
      if (k0 + 32 * kc >= kend) break;  // wave-uniform
#pragma unroll
      for (int rb = 0; rb < GT; ++rb)
#pragma unroll
        for (int cb = 0; cb < GT; ++cb)
          acc[rb][cb] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[kc][rb], y[kc][cb], acc[rb][cb], 0, 0, 0);
    }
  }
  float* part = a.part[q] + (int64_t)split * a.in_dim[q] * a.out_dim[q];
#pragma unroll
  for (int rb = 0; rb < GT; ++rb)
#pragma unroll
    for (int cb = 0; cb < GT; ++cb)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        part[(int64_t)(m0 + rb * 16 + (l >> 4) * 4 + j) * a.out_dim[q] + n0 + cb * 16 + lr] =
            acc[rb][cb][j];
}

__global__ __launch_bounds__(256) void grad_kernel(const GradArgs a) {
  __shared__ float red[4];
  // (the wave's number as a scalar: the layer's tables are read once, by it)
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  // the batch chunks of an XCD's workgroups are its own (workgroups go to the
  // XCDs in turn): an XCD reads an eighth of the batch, not all of it
  const int n_tiles = a.first_tile[4], tile_blocks = GRAD_XCDS * grad_blocks(n_tiles);
  if ((int)blockIdx.x < tile_blocks) {
    const int t = 4 * ((int)blockIdx.x / GRAD_XCDS) + wave, i = t / n_tiles;
    if (i < MLP_SPLITK / GRAD_XCDS)
      weight_grad_tile(a, t - i * n_tiles,
                       (int)blockIdx.x % GRAD_XCDS * (MLP_SPLITK / GRAD_XCDS) + i, l);
    return;
  }
  const int c = (int)blockIdx.x - tile_blocks;
  int q = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i) q = c >= a.first_col[i] ? i : q;
  const int n = c - a.first_col[q];
  const bf16* row = a.dZt[q] + (int64_t)n * a.cap;
  float s = 0.f;
  for (int64_t m = (int64_t)threadIdx.x * 8; m < a.M; m += 256 * 8) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(row + m);
#pragma unroll
    for (int k = 0; k < 8; ++k) s += (float)v[k];
  }
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (l == 0) red[wave] = s;
  __syncthreads();
  if (threadIdx.x == 0) a.grad_b[q][n] = (red[0] + red[1]) + (red[2] + red[3]);
}

struct AdamArgs {
  float* master;
  float* m;
  float* v;
  float* grad;
  const float* part[4];
  bf16* Wt[4];
  bf16* Wk[4];
  int64_t oW[4], ob[4];
  int in_dim[4], out_dim[4];
  int first_tile[5];  // first tile of each layer's weights; then the total
  int first_col[5];   // first bias of each layer; then the total
  float lr, beta1, beta2, eps, bc1, bc2;
  int update;  // 0: only assemble the gradient
};

__device__ __forceinline__ float adam_update(const AdamArgs& a, int64_t i, float g) {
  const float m = a.beta1 * a.m[i] + (1.f - a.beta1) * g;
  const float v = a.beta2 * a.v[i] + (1.f - a.beta2) * g * g;
  a.m[i] = m;
  a.v[i] = v;
  const float w = a.master[i] - a.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.eps);
  a.master[i] = w;
  return w;
}

// A workgroup per 8 x 32 tile of a layer's weights (ADAM_K inputs, ADAM_N
// outputs, so that the transposed bfloat16 copy goes out in 16-byte pieces
// instead of single values), then one per 256 biases.
constexpr int ADAM_K = 8, ADAM_N = 32;
__global__ __launch_bounds__(256) void adam_kernel(const AdamArgs a) {
  __shared__ __align__(16) bf16 wt[ADAM_N * ADAM_K];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (b >= a.first_tile[4]) {
    const int c = (b - a.first_tile[4]) * 256 + tid;
    if (c >= a.first_col[4] || !a.update) return;
    int64_t i = a.ob[0] + c;
#pragma unroll
    for (int q = 1; q < 4; ++q) i = c >= a.first_col[q] ? a.ob[q] + (c - a.first_col[q]) : i;
    adam_update(a, i, a.grad[i]);  // (written by grad_kernel)
    return;
  }
  int q = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i) q = b >= a.first_tile[i] ? i : q;
  const int t = b - a.first_tile[q], in = a.in_dim[q], out = a.out_dim[q], nn = out / ADAM_N;
  const int k = t / nn * ADAM_K + tid / ADAM_N, n = t % nn * ADAM_N + tid % ADAM_N;
  const int64_t e = (int64_t)k * out + n, i = a.oW[q] + e;
  const float* part = a.part[q] + e;
  float x[MLP_SPLITK], g = 0.f;
#pragma unroll
  for (int s = 0; s < MLP_SPLITK; ++s) x[s] = part[(int64_t)s * in * out];
#pragma unroll
  for (int s = 0; s < MLP_SPLITK; ++s) g += x[s];
  a.grad[i] = g;
  if (!a.update) return;
  const float w = adam_update(a, i, g);
  a.Wk[q][e] = (bf16)w;
  wt[(tid % ADAM_N) * ADAM_K + tid / ADAM_N] = (bf16)w;
  __syncthreads();
  if (tid < ADAM_N)
    *(bf16x8*)(a.Wt[q] + (int64_t)(t % nn * ADAM_N + tid) * in + t / nn * ADAM_K) =
        *(const bf16x8*)(wt + tid * ADAM_K);
}

struct RefreshArgs {
  const float* master;
  bf16* Wt[4];
  bf16* Wk[4];
  int64_t oW[4];
  int in_dim[4], out_dim[4];
};

__global__ void refresh_kernel(const RefreshArgs a, int l) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)a.in_dim[l] * a.out_dim[l]) return;
  const int k = (int)(e / a.out_dim[l]);
  const int n = (int)(e - (int64_t)k * a.out_dim[l]);
  const bf16 w = (bf16)a.master[a.oW[l] + e];
  a.Wt[l][(int64_t)n * a.in_dim[l] + k] = w;
  a.Wk[l][e] = w;
}

// Network outputs -> model parameters (the field vector is encoded as
// (B cos g, B sin g cos 2psi, B sin g sin 2psi) / 3000), then the box.
__device__ __forceinline__ void decode_row(const float* y_in, const float* __restrict__ out_mean,
                                           const float* __restrict__ out_std, float* codes,
                                           float* params) {
  float y[MLP_NCODE];
#pragma unroll
  for (int c = 0; c < MLP_NCODE; ++c) y[c] = y_in[c];
  if (codes) {
#pragma unroll
    for (int c = 0; c < MLP_NCODE; ++c) codes[c] = y[c];
  }
  if (!params) return;
  double P[NPAR];
  const double bt = sqrt((double)y[1] * y[1] + (double)y[2] * y[2]);
  P[0] = 3000.0 * sqrt((double)y[0] * y[0] + bt * bt);
  P[1] = atan2(bt, (double)y[0]) * (180.0 / 3.14159265358979323846);
  P[2] = 0.5 * atan2((double)y[2], (double)y[1]) * (180.0 / 3.14159265358979323846);
#pragma unroll
  for (int c = 3; c < MLP_NCODE; ++c) P[c] = (double)y[c] * out_std[c - 3] + out_mean[c - 3];
  project(P);
#pragma unroll
  for (int c = 0; c < NPAR; ++c) params[c] = (float)P[c];
}

// ---- fused inference ---------------------------------------------------------
// One workgroup of four waves carries FT rows through the whole network:
// standardised inputs and hidden activations stay in one LDS tile
// (bfloat16, rows padded by 8 elements so that the 16 rows an MFMA operand
// reads fall in different banks; each layer finishes reading the tile before
// any wave overwrites it with the layer's outputs), weights are read as MFMA
// operands from L2, and the outputs are decoded in place.  Wave w owns
// hidden columns [64 w, 64 w + 64) and output rows [16 w, 16 w + 16).
// (128-row tiles would halve the weight reads but need 335 registers per
// lane, one wave per SIMD: measured 1.5x slower.)  The MFMA sequence per
// output element (same instruction, same k order, same epilogue) is that of
// the training step's forward pass, so the results are equal.
constexpr int FT = 64;
// waves per inference workgroup; each owns IW_COLS of a hidden layer's 256
// columns for the tile's 64 rows (eight waves keep the registers per wave
// low enough for four waves per SIMD, which hide the weight loads' latency)
constexpr int IW = 8;
constexpr int IW_CB = MLP_H / (16 * IW);  // 16-column MFMA tiles per wave

struct MlpInferArgs {
  const float* stokes;
  int64_t M;
  int n_in, K0;
  const float* mean;
  const float* istd;
  const bf16* Wt[4];
  const float* bias[4];
  const float* out_mean;
  const float* out_std;
  float* codes;
  float* params;
};

template <int KS>
__device__ __forceinline__ void fused_hidden(bf16* buf, int ldin, int Kd, const bf16* W,
                                             const float* __restrict__ bias, int wave, int l) {
  const bf16* in = buf;
  const int K = KS > 0 ? KS : Kd;
  const int lr = l & 15, lk = (l >> 4) * 8;
  f32x4 acc[4][IW_CB];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < IW_CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bf16* wrow = W + (int64_t)(wave * 16 * IW_CB + lr) * K + lk;
  auto mfma_step = [&](const bf16x8 (&b)[IW_CB], int k) {
    bf16x8 a[4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) a[rb] = *(const bf16x8*)(in + (rb * 16 + lr) * ldin + k + lk);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < IW_CB; ++cb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rb], b[cb], acc[rb][cb], 0, 0, 0);
  };
  if constexpr (KS > 0) {
    // the weights (read from L2 by every row tile) two k-steps ahead of
    // their MFMAs
    constexpr int NK = KS / 32, PF = 2;
    bf16x8 b[NK][IW_CB];
#pragma unroll
    for (int s = 0; s < NK; ++s) {
      if (s == 0) {
#pragma unroll
        for (int q = 0; q < PF && q < NK; ++q)
#pragma unroll
          for (int cb = 0; cb < IW_CB; ++cb)
            b[q][cb] = *(const bf16x8*)(wrow + (int64_t)cb * 16 * K + 32 * q);
      }
      if (s + PF < NK) {
#pragma unroll
        for (int cb = 0; cb < IW_CB; ++cb)
          b[s + PF][cb] = *(const bf16x8*)(wrow + (int64_t)cb * 16 * K + 32 * (s + PF));
      }
      mfma_step(b[s], 32 * s);
    }
  } else {
    for (int k = 0; k < K; k += 32) {
      bf16x8 b[IW_CB];
#pragma unroll
      for (int cb = 0; cb < IW_CB; ++cb) b[cb] = *(const bf16x8*)(wrow + (int64_t)cb * 16 * K + k);
      mfma_step(b, k);
    }
  }
  __syncthreads();  // every wave has read the layer's inputs
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < IW_CB; ++cb)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = rb * 16 + (l >> 4) * 4 + j;
        const int col = wave * 16 * IW_CB + cb * 16 + lr;
        buf[row * LDH + col] = (bf16)gelu(acc[rb][cb][j] + bias[col]);
      }
  __syncthreads();
}

__global__ __launch_bounds__(IW * 64) void mlp_infer_kernel(const MlpInferArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int ldx = a.K0 + 8;
  bf16* buf = (bf16*)smem;  // [FT][max(K0 + 8, LDH)]
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int64_t row0 = (int64_t)blockIdx.x * FT;
  for (int idx = tid; idx < FT * a.K0; idx += IW * 64) {
    const int r = idx / a.K0, k = idx - r * a.K0;
    const int64_t row = row0 + r;
    float x = 0.f;
    if (k < a.n_in && row < a.M) x = (a.stokes[row * a.n_in + k] - a.mean[k]) * a.istd[k];
    buf[r * ldx + k] = (bf16)x;
  }
  __syncthreads();
  fused_hidden<0>(buf, ldx, a.K0, a.Wt[0], a.bias[0], wave, l);
  fused_hidden<MLP_H>(buf, LDH, MLP_H, a.Wt[1], a.bias[1], wave, l);
  fused_hidden<MLP_H>(buf, LDH, MLP_H, a.Wt[2], a.bias[2], wave, l);
  float* y4 = (float*)smem;  // [FT][MLP_OUT + 1], over the tile once it is read
  {  // output layer: waves 0-3 take rows [16 wave, 16 wave + 16), 32 columns
    const int lr = l & 15, lk = (l >> 4) * 8;
    const bool mine = wave < FT / 16;  // wave-uniform
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    if (mine) {
#pragma unroll
      for (int k = 0; k < MLP_H; k += 32) {
        const bf16x8 av = *(const bf16x8*)(buf + (wave * 16 + lr) * LDH + k + lk);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const bf16x8 bv = *(const bf16x8*)(a.Wt[3] + (int64_t)(cb * 16 + lr) * MLP_H + k + lk);
          acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[cb], 0, 0, 0);
        }
      }
    }
    __syncthreads();  // the tile is read; its space takes the outputs
    if (mine) {
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int row = wave * 16 + (l >> 4) * 4 + j;
          const int col = cb * 16 + lr;
          y4[row * (MLP_OUT + 1) + col] = acc[cb][j] + a.bias[3][col];
        }
    }
  }
  __syncthreads();
  if (tid < FT) {
    const int64_t row = row0 + tid;
    if (row < a.M)
      decode_row(&y4[tid * (MLP_OUT + 1)], a.out_mean, a.out_std,
                 a.codes ? a.codes + row * MLP_NCODE : nullptr,
                 a.params ? a.params + row * NPAR : nullptr);
  }
}

// Networks with at most 32 inputs (the HMI filtergrams: one k-step in the
// first layer): a persistent grid of one 8-wave workgroup per CU whose waves
// keep their columns' weights of the two 256 x 256 layers in registers
// (128 per lane) and walk the 64-row tiles, so the weights are read from L2 once per
// workgroup instead of once per tile.  The tile and the per-element MFMA
// sequence (same instruction, same k order) are those of mlp_infer_kernel,
// with the hidden layers' operands swapped (the output transposed, so that
// a lane's four results are consecutive columns of one row: one 8-byte LDS
// write instead of four 2-byte ones; each element is the same dot product);
// the hidden layers' GELU comes from a table (below), so an activation may
// differ from mlp_infer_kernel's in its last bfloat16 bit where its value
// lies within 6e-7 of a rounding midpoint.  Output layer: wave w takes rows
// [16 (w / 2), 16 (w / 2) + 16) and columns [16 (w % 2), +16).
// GELU by linear interpolation in a table of GELU at z = -6 + i / 512
// (i < 6144, each entry {GELU(z_i), GELU(z_i+1) - GELU(z_i)}, built in LDS by
// each workgroup from gelu()): interpolation error below (1/512)^2 / 8 times
// max |GELU''| = 0.8, i.e. 4e-7, on top of gelu()'s 1.5e-7, against
// 2^-9 relative for the bfloat16 the result is stored in; above z = 6
// GELU(z) = z to 6e-9, below -6 the first entry (-6e-9) stands for ~0.
// About ten vector instructions instead of gelu()'s thirteen plus two
// transcendental ones, in the epilogue that bounds the resident kernel.
constexpr int GELU_TAB_N = 6144;
__device__ __forceinline__ float gelu_tab(const float2* __restrict__ tab, float z) {
  const float x = fminf(fmaxf(fmaf(z, 512.f, 3072.f), 0.f), (float)(GELU_TAB_N - 1));
  const float i = floorf(x);
  const float2 e = tab[(int)i];
  const float g = fmaf(x - i, e.y, e.x);
  return z >= 6.f ? z : g;
}

__device__ __forceinline__ void resident_hidden_epilogue(bf16* buf, const f32x4 (&acc)[4][IW_CB],
                                                         const float* __restrict__ bias,
                                                         const float2* __restrict__ tab, int wave,
                                                         int l) {
  typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
#pragma unroll
  for (int cb = 0; cb < IW_CB; ++cb) {
    const int col0 = wave * 16 * IW_CB + cb * 16 + (l >> 4) * 4;
    const float4 b4 = *reinterpret_cast<const float4*>(bias + col0);
    const float bb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const int row = rb * 16 + (l & 15);
      bf16x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (bf16)gelu_tab(tab, acc[rb][cb][j] + bb[j]);
      *reinterpret_cast<bf16x4*>(buf + row * LDH + col0) = v;
    }
  }
}

// The layer as D^T = W X^T: the weights are the A operand and the tile's
// rows the B operand, so that lane l receives four consecutive output
// columns of one row and stores them with one 8-byte write.
template <int NK>
__device__ __forceinline__ void resident_hidden(bf16* buf, int ldin, const bf16x8 (&w)[NK][IW_CB],
                                                const float* __restrict__ bias,
                                                const float2* __restrict__ tab, int wave, int l) {
  const int lr = l & 15, lk = (l >> 4) * 8;
  f32x4 acc[4][IW_CB];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
#pragma unroll
    for (int cb = 0; cb < IW_CB; ++cb) acc[rb][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NK; ++s) {
    bf16x8 av[4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
      av[rb] = *(const bf16x8*)(buf + (rb * 16 + lr) * ldin + 32 * s + lk);
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int cb = 0; cb < IW_CB; ++cb)
        acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s][cb], av[rb], acc[rb][cb], 0, 0, 0);
  }
  __syncthreads();  // every wave has read the layer's inputs
  resident_hidden_epilogue(buf, acc, bias, tab, wave, l);
  __syncthreads();
}

static_assert(IW == 8 && IW_CB == 2, "the resident kernel's output split assumes 8 waves");
// LDS of the resident kernel: the 64-row tile (or the outputs over it), then
// the GELU table
constexpr size_t RESIDENT_TAB_OFFSET = sizeof(bf16) * FT * LDH;
constexpr size_t RESIDENT_LDS = RESIDENT_TAB_OFFSET + sizeof(float2) * GELU_TAB_N;
static_assert(sizeof(float) * FT * (MLP_OUT + 1) <= RESIDENT_TAB_OFFSET && RESIDENT_TAB_OFFSET % 16 == 0,
              "the outputs fit over the tile");

__global__ __launch_bounds__(IW * 64, 1) void mlp_infer_resident_kernel(const MlpInferArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int K0 = 32, NKH = MLP_H / 32;
  constexpr int ldx = K0 + 8;
  bf16* buf = (bf16*)smem;  // [FT][LDH]
  float* y4 = (float*)smem;  // [FT][MLP_OUT + 1], over the tile once it is read
  float2* tab = (float2*)(smem + RESIDENT_TAB_OFFSET);  // [GELU_TAB_N]
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int lr = l & 15, lk = (l >> 4) * 8;
  for (int i = tid; i < GELU_TAB_N; i += IW * 64) {
    const float z0 = -6.f + (float)i * (1.f / 512.f), z1 = -6.f + (float)(i + 1) * (1.f / 512.f);
    const float g0 = gelu(z0);
    tab[i] = make_float2(g0, gelu(z1) - g0);
  }
  // (the table is complete before the first epilogue: the first tile's
  // input barrier comes first)
  // this wave's columns of every layer, as MFMA B fragments
  // (hidden layers 1 and 2: 128 registers; the small first and output
  // layers are read through the caches at each tile)
  bf16x8 w1[NKH][IW_CB], w2[NKH][IW_CB];
#pragma unroll
  for (int cb = 0; cb < IW_CB; ++cb) {
    const int col = wave * 16 * IW_CB + cb * 16 + lr;
#pragma unroll
    for (int s = 0; s < NKH; ++s) {
      w1[s][cb] = *(const bf16x8*)(a.Wt[1] + (int64_t)col * MLP_H + 32 * s + lk);
      w2[s][cb] = *(const bf16x8*)(a.Wt[2] + (int64_t)col * MLP_H + 32 * s + lk);
    }
  }
  const int orb = wave >> 1, ocb = wave & 1;  // output-layer block of this wave
  const int64_t n_tiles = (a.M + FT - 1) / FT;
  // the inputs of the workgroup's next tile are loaded into registers while
  // the current one is computed (4 values per lane), so that their latency
  // is not exposed between the tiles
  constexpr int NXL = FT * K0 / (IW * 64);
  static_assert(NXL * IW * 64 == FT * K0, "whole input tiles");
  float xin[NXL];
  auto load_inputs = [&](int64_t t) {
#pragma unroll
    for (int q = 0; q < NXL; ++q) {
      const int idx = tid + q * IW * 64;
      const int r = idx / K0, k = idx - r * K0;
      const int64_t row = t * FT + r;
      xin[q] = (k < a.n_in && row < a.M) ? a.stokes[row * a.n_in + k] : 0.f;
    }
  };
  if (blockIdx.x < n_tiles) load_inputs(blockIdx.x);
  for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const int64_t row0 = tile * FT;
#pragma unroll
    for (int q = 0; q < NXL; ++q) {
      const int idx = tid + q * IW * 64;
      const int r = idx / K0, k = idx - r * K0;
      buf[r * ldx + k] = (bf16)(k < a.n_in ? (xin[q] - a.mean[k]) * a.istd[k] : 0.f);
    }
    if (tile + gridDim.x < n_tiles) load_inputs(tile + gridDim.x);
    bf16x8 w0[1][IW_CB];
#pragma unroll
    for (int cb = 0; cb < IW_CB; ++cb)
      w0[0][cb] = *(const bf16x8*)(a.Wt[0] + (int64_t)(wave * 16 * IW_CB + cb * 16 + lr) * K0 + lk);
    __syncthreads();
    resident_hidden<1>(buf, ldx, w0, a.bias[0], tab, wave, l);
    resident_hidden<NKH>(buf, LDH, w1, a.bias[1], tab, wave, l);
    resident_hidden<NKH>(buf, LDH, w2, a.bias[2], tab, wave, l);
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NKH; ++s) {
      const bf16x8 av = *(const bf16x8*)(buf + (orb * 16 + lr) * LDH + 32 * s + lk);
      const bf16x8 wv = *(const bf16x8*)(a.Wt[3] + (int64_t)(ocb * 16 + lr) * MLP_H + 32 * s + lk);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, wv, acc, 0, 0, 0);
    }
    __syncthreads();  // the tile is read; its space takes the outputs
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = orb * 16 + (l >> 4) * 4 + j;
      y4[row * (MLP_OUT + 1) + ocb * 16 + lr] = acc[j] + a.bias[3][ocb * 16 + lr];
    }
    __syncthreads();
    if (tid < FT) {
      const int64_t row = row0 + tid;
      if (row < a.M)
        decode_row(&y4[tid * (MLP_OUT + 1)], a.out_mean, a.out_std,
                   a.codes ? a.codes + row * MLP_NCODE : nullptr,
                   a.params ? a.params + row * NPAR : nullptr);
    }
    __syncthreads();  // the outputs are read before the next tile's inputs
  }
}

static_assert(MLP_MAX_IN % 32 == 0 && FT * (MLP_MAX_IN + 8) * 2 <= MLP_LDS_MAX,
              "the widest input must fit a tile");

size_t mlp_infer_lds_bytes(int K0) {
  const int ldx = K0 + 8, ld = ldx > LDH ? ldx : LDH;
  const size_t tile = sizeof(bf16) * (size_t)FT * ld;
  const size_t outs = sizeof(float) * FT * (MLP_OUT + 1);
  return tile > outs ? tile : outs;
}

hipError_t mlp_infer(const MlpDev& net, int64_t M, const float* stokes, float* codes,
                     float* params, hipStream_t s) {
  const MlpLayout& L = net.L;
  MlpInferArgs a;
  a.stokes = stokes;
  a.M = M;
  a.n_in = L.n_in;
  a.K0 = L.K0;
  a.mean = net.in_mean;
  a.istd = net.in_istd;
  for (int l = 0; l < 4; ++l) {
    a.Wt[l] = net.Wt[l];
    a.bias[l] = net.master + L.ob[l];
  }
  a.out_mean = net.out_mean;
  a.out_std = net.out_std;
  a.codes = codes;
  a.params = params;
  // tiles of wide inputs exceed the 64 KB default of dynamic LDS and need
  // the kernel attribute (gfx950 has 160 KB per workgroup); set once per
  // process, before the first launch (not a stream operation)
  static const hipError_t attr = hipFuncSetAttribute(
      (const void*)mlp_infer_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, MLP_LDS_MAX);
  if (attr != hipSuccess) return attr;
  const size_t lds = mlp_infer_lds_bytes(L.K0);
  const int64_t tiles = (M + FT - 1) / FT;
  if (tiles < 1) return hipSuccess;
  if (L.K0 == 32) {
    // one workgroup per CU (the CU count of this device, queried once)
    static int cus[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (cus[dev] == 0) {
      int v = 0;
      e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
      if (e != hipSuccess) return e;
      cus[dev] = v > 0 ? v : 1;
    }
    static const hipError_t rattr =
        hipFuncSetAttribute((const void*)mlp_infer_resident_kernel,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)RESIDENT_LDS);
    if (rattr != hipSuccess) return rattr;
    const int64_t grid = tiles < cus[dev] ? tiles : cus[dev];
    mlp_infer_resident_kernel<<<(unsigned)grid, IW * 64, RESIDENT_LDS, s>>>(a);
    return hipGetLastError();
  }
  mlp_infer_kernel<<<(unsigned)tiles, IW * 64, lds, s>>>(a);
  return hipGetLastError();
}

// Pixels whose fit is not acceptable go to the list.  Each block takes a
// contiguous chunk of SELECT_PER_THREAD * 256 pixels, ranks its selections
// with a block-wide scan in LDS and reserves its slots with one atomic, so
// the counter sees one update per 4096 pixels (same-address atomics
// serialise in L2).
constexpr int SELECT_PER_THREAD = 16;
__global__ __launch_bounds__(256) void fallback_select_kernel(const double* __restrict__ chi2,
                                                              const int32_t* __restrict__ status,
                                                              int64_t n, double tau,
                                                              int unconverged, int32_t* list,
                                                              unsigned long long* count) {
  __shared__ unsigned int scan[256];
  __shared__ unsigned long long base;
  const int t = threadIdx.x;
  const int64_t start = (int64_t)blockIdx.x * 256 * SELECT_PER_THREAD;
  unsigned int mask = 0u, c = 0u;
#pragma unroll
  for (int k = 0; k < SELECT_PER_THREAD; ++k) {
    const int64_t i = start + (int64_t)k * 256 + t;
    if (i < n) {
      const double v = chi2[i];
      bool sel = !(v <= tau) && !isnan(v);  // not acceptable (non-finite input stays as is)
      if (unconverged && !isnan(v)) {
        const int code = status[i] & 15;
        sel = sel || (code != 0 && code != 3);
      }
      if (sel) {
        mask |= 1u << k;
        ++c;
      }
    }
  }
  scan[t] = c;
  __syncthreads();
  // inclusive Hillis-Steele scan over the 256 counts
  for (int off = 1; off < 256; off <<= 1) {
    const unsigned int v = t >= off ? scan[t - off] : 0u;
    __syncthreads();
    scan[t] += v;
    __syncthreads();
  }
  if (t == 255) base = scan[255] ? atomicAdd(count, (unsigned long long)scan[255]) : 0ull;
  __syncthreads();
  unsigned long long pos = base + scan[t] - c;
#pragma unroll
  for (int k = 0; k < SELECT_PER_THREAD; ++k)
    if (mask & (1u << k)) list[pos++] = (int32_t)(start + (int64_t)k * 256 + t);
}

__global__ void fallback_merge_kernel(const int32_t* __restrict__ list,
                                      const unsigned long long* __restrict__ count,
                                      const float* __restrict__ p_fb,
                                      const double* __restrict__ c_fb,
                                      const int32_t* __restrict__ i_fb,
                                      const int32_t* __restrict__ s_fb, int keep_refit,
                                      float* params, double* chi2, int32_t* iters,
                                      int32_t* status) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if ((unsigned long long)t >= *count) return;
  const int64_t i = list[t];
  const bool better = keep_refit || c_fb[i] < chi2[i];
  if (better) {
#pragma unroll
    for (int q = 0; q < NPAR; ++q) params[i * NPAR + q] = p_fb[i * NPAR + q];
    chi2[i] = c_fb[i];
  }
  iters[i] += i_fb[i];
  if (status) status[i] = (better ? s_fb[i] : status[i]) | 16;
}

// ---- host-side sequences ---------------------------------------------------

static unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

__global__ void copy_u64_kernel(unsigned long long* dst, const unsigned long long* src, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    dst[i] = src[i];
}

hipError_t copy_u64(unsigned long long* dst, const unsigned long long* src, int n, hipStream_t s) {
  copy_u64_kernel<<<1, 64, 0, s>>>(dst, src, n);
  return hipGetLastError();
}

__global__ void zero_u64_kernel(unsigned long long* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

hipError_t zero_u64(unsigned long long* p, int n, hipStream_t s) {
  zero_u64_kernel<<<blocks_for(n, 64), 64, 0, s>>>(p, n);
  return hipGetLastError();
}

// ---- training-set preparation --------------------------------------------

// Each block takes MOM_ROWS consecutive rows.  With fewer than 256 columns
// thread t owns column t % ncols and every (256 / ncols)-th row from
// t / ncols, so that consecutive threads read consecutive elements; with
// more, thread t owns columns t, t + 256, ...  Sums stay in registers, then
// go to LDS and to the global float64 accumulators once per block.
constexpr int MOM_ROWS = 2048;

__global__ __launch_bounds__(256) void col_moments_kernel(const float* __restrict__ X, int64_t n,
                                                          int ld, int col0, int ncols,
                                                          double* sums) {
  extern __shared__ double acc[];  // [2 * ncols]
  const int t = threadIdx.x;
  for (int c = t; c < 2 * ncols; c += blockDim.x) acc[c] = 0.0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * MOM_ROWS;
  const int rows = (int)(n - r0 < MOM_ROWS ? n - r0 : MOM_ROWS);
  if (ncols < 256) {
    const int tpc = 256 / ncols;
    if (t < tpc * ncols) {
      const int c = t % ncols;
      double s1 = 0.0, s2 = 0.0;
      for (int r = t / ncols; r < rows; r += tpc) {
        const double x = (double)X[(r0 + r) * ld + col0 + c];
        s1 += x;
        s2 += x * x;
      }
      atomicAdd(&acc[2 * c], s1);
      atomicAdd(&acc[2 * c + 1], s2);
    }
  } else {
    for (int c = t; c < ncols; c += 256) {
      double s1 = 0.0, s2 = 0.0;
      for (int r = 0; r < rows; ++r) {
        const double x = (double)X[(r0 + r) * ld + col0 + c];
        s1 += x;
        s2 += x * x;
      }
      acc[2 * c] += s1;  // this thread alone owns column c
      acc[2 * c + 1] += s2;
    }
  }
  __syncthreads();
  for (int c = t; c < 2 * ncols; c += blockDim.x) atomicAdd(&sums[c], acc[c]);
}

hipError_t col_moments(const float* X, int64_t n, int ld, int col0, int ncols, double* sums,
                       hipStream_t s) {
  if (n <= 0) return hipSuccess;
  col_moments_kernel<<<blocks_for(n, MOM_ROWS), 256, sizeof(double) * 2 * ncols, s>>>(
      X, n, ld, col0, ncols, sums);
  return hipGetLastError();
}

__global__ void encode_targets_kernel(const float* __restrict__ P, int64_t n,
                                      const float* __restrict__ out_mean,
                                      const float* __restrict__ out_std, float* T) {
  const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= n) return;
  const float* p = P + m * NPAR;
  float* t = T + m * MLP_NCODE;
  const float g = p[1] * (float)(3.14159265358979323846 / 180.0);
  const float p2 = p[2] * (float)(3.14159265358979323846 / 90.0);
  const float b = p[0] * (1.f / 3000.f);
  t[0] = b * cosf(g);
  t[1] = b * sinf(g) * cosf(p2);
  t[2] = b * sinf(g) * sinf(p2);
#pragma unroll
  for (int c = 3; c < MLP_NCODE; ++c) t[c] = (p[c] - out_mean[c - 3]) / out_std[c - 3];
}

hipError_t encode_targets(const float* P, int64_t n, const float* out_mean, const float* out_std,
                          float* T, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  encode_targets_kernel<<<blocks_for(n, 256), 256, 0, s>>>(P, n, out_mean, out_std, T);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void sq_diff_sum_kernel(const float* __restrict__ A,
                                                          const float* __restrict__ B,
                                                          int64_t count, double* out) {
  __shared__ double red[256];
  double v = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double d = (double)A[i] - (double)B[i];
    v += d * d;
  }
  red[threadIdx.x] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(out, red[0]);
}

hipError_t sq_diff_sum(const float* A, const float* B, int64_t count, double* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const int64_t blocks = (count + 255) / 256;
  sq_diff_sum_kernel<<<(unsigned)(blocks < 4096 ? blocks : 4096), 256, 0, s>>>(A, B, count, out);
  return hipGetLastError();
}

template <int RB>
static hipError_t launch_train_rows(const TrainRowsArgs& a, hipStream_t s) {
  const size_t lds = train_lds_bytes<RB>(a.K0);
  hipError_t e = hipSuccess;
  if (lds > 64 * 1024)
    e = hipFuncSetAttribute((const void*)train_rows_kernel<RB>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, MLP_LDS_MAX);
  if (e != hipSuccess) return e;
  train_rows_kernel<RB><<<blocks_for(a.M, 16 * RB), TW * 64, lds, s>>>(a);
  return hipGetLastError();
}
static_assert(train_lds_bytes<2>((MLP_MAX_IN + 31) / 32 * 32) <= MLP_LDS_MAX, "the rows' LDS");

hipError_t mlp_pass(const MlpDev& net, MlpWork& w, int64_t M, const float* stokes,
                    const float* targets, const int32_t* rows, hipStream_t s) {
  const MlpLayout& L = net.L;
  TrainRowsArgs a;
  a.stokes = stokes;
  a.rows = rows;
  a.targets = targets;
  a.M = M;
  a.cap = w.cap;
  a.n_in = L.n_in;
  a.K0 = L.K0;
  a.mean = net.in_mean;
  a.istd = net.in_istd;
  a.X0t = w.X0t;
  a.loss = w.loss;
  GradArgs g;
  g.M = M;
  g.cap = w.cap;
  g.chunk = ((M + MLP_SPLITK - 1) / MLP_SPLITK + 31) / 32 * 32;
  int64_t off = 0;
  int tiles = 0, cols = 0;
  for (int l = 0; l < 4; ++l) {
    a.Wt[l] = net.Wt[l];
    a.Wk[l] = net.Wk[l];
    a.bias[l] = net.master + L.ob[l];
    a.dZt[l] = w.dZt[l];
    if (l < 3) a.Yt[l] = w.Yt[l];
    g.Xt[l] = l == 0 ? w.X0t : w.Yt[l - 1];
    g.dZt[l] = w.dZt[l];
    g.part[l] = w.dW + off;
    g.grad_b[l] = w.grad + L.ob[l];
    g.in_dim[l] = L.in_dim[l];
    g.out_dim[l] = L.out_dim[l];
    g.first_tile[l] = tiles;
    g.first_col[l] = cols;
    off += (int64_t)L.in_dim[l] * L.out_dim[l] * MLP_SPLITK;
    tiles += L.in_dim[l] / (16 * GT) * (L.out_dim[l] / (16 * GT));
    cols += L.out_dim[l];
  }
  g.first_tile[4] = tiles;
  g.first_col[4] = cols;
  const hipError_t e = M >= TRAIN_RB2_ROWS ? launch_train_rows<2>(a, s) : launch_train_rows<1>(a, s);
  if (e != hipSuccess) return e;
  grad_kernel<<<GRAD_XCDS * grad_blocks(tiles) + cols, 256, 0, s>>>(g);
  return hipGetLastError();
}

hipError_t mlp_adam(const MlpDev& net, const MlpWork& w, float lr, float beta1, float beta2,
                    float eps, int step, hipStream_t s) {
  const MlpLayout& L = net.L;
  AdamArgs a;
  a.master = net.master;
  a.m = net.adam_m;
  a.v = net.adam_v;
  a.grad = w.grad;
  int64_t off = 0;
  int tiles = 0, cols = 0;
  for (int l = 0; l < 4; ++l) {
    a.part[l] = w.dW + off;
    off += (int64_t)L.in_dim[l] * L.out_dim[l] * MLP_SPLITK;
    a.Wt[l] = net.Wt[l];
    a.Wk[l] = net.Wk[l];
    a.oW[l] = L.oW[l];
    a.ob[l] = L.ob[l];
    a.in_dim[l] = L.in_dim[l];
    a.out_dim[l] = L.out_dim[l];
    a.first_tile[l] = tiles;
    a.first_col[l] = cols;
    tiles += L.in_dim[l] / ADAM_K * (L.out_dim[l] / ADAM_N);
    cols += L.out_dim[l];
  }
  a.first_tile[4] = tiles;
  a.first_col[4] = cols;
  a.lr = lr;
  a.beta1 = beta1;
  a.beta2 = beta2;
  a.eps = eps;
  a.update = step > 0 ? 1 : 0;
  a.bc1 = step > 0 ? 1.f - powf(beta1, (float)step) : 1.f;
  a.bc2 = step > 0 ? 1.f - powf(beta2, (float)step) : 1.f;
  adam_kernel<<<tiles + blocks_for(cols, 256), 256, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t mlp_refresh_bf16(const MlpDev& net, hipStream_t s) {
  RefreshArgs r;
  r.master = net.master;
  for (int l = 0; l < 4; ++l) {
    r.Wt[l] = net.Wt[l];
    r.Wk[l] = net.Wk[l];
    r.oW[l] = net.L.oW[l];
    r.in_dim[l] = net.L.in_dim[l];
    r.out_dim[l] = net.L.out_dim[l];
  }
  for (int l = 0; l < 4; ++l) {
    const int64_t n = (int64_t)net.L.in_dim[l] * net.L.out_dim[l];
    refresh_kernel<<<blocks_for(n, 256), 256, 0, s>>>(r, l);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t fallback_select(const double* chi2, const int32_t* status, int64_t n, double tau,
                           bool unconverged, int32_t* list, unsigned long long* count,
                           hipStream_t s) {
  if (unconverged && !status) return hipErrorInvalidValue;
  fallback_select_kernel<<<blocks_for(n, 256 * SELECT_PER_THREAD), 256, 0, s>>>(
      chi2, status, n, tau, unconverged ? 1 : 0, list, count);
  return hipGetLastError();
}

hipError_t fallback_merge(const int32_t* list, const unsigned long long* count, int64_t n,
                          const float* p_fb, const double* c_fb, const int32_t* i_fb,
                          const int32_t* s_fb, bool keep_refit, float* params, double* chi2,
                          int32_t* iters, int32_t* status, hipStream_t s) {
  fallback_merge_kernel<<<blocks_for(n, 256), 256, 0, s>>>(
      list, count, p_fb, c_fb, i_fb, s_fb, keep_refit ? 1 : 0, params, chi2, iters, status);
  return hipGetLastError();
}

}  // namespace vfisv
