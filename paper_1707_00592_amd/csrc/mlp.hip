// Learned nonlinear weights: training data, bf16 MFMA forward/backward,
// Adam, and packing for the stage kernel (isweno_mlp_*).
#include <hip/hip_runtime.h>

#include "ctx.hpp"
#include "isweno.h"
#include "mlp.hpp"
#include "sweep.hpp"

namespace isw {

constexpr int MLP_WAVES = 4;   // waves per workgroup of the forward kernel
constexpr int GRAD_WAVES = 8;  // and of the gradient (one workgroup a CU at 65 536 samples)

// Scale of the value error in the loss and tolerance of the confidence
// label, in units of the stencil's range (the inputs are normalised to it).
constexpr float kValueScale = 0.01f;
constexpr float kConfTol = 0.005f;

// Candidates of eq. (20) on a normalised stencil a..e = v_{i-2}..v_{i+2}.
__device__ __forceinline__ void candidates(float a, float b, float c, float d, float e,
                                           float* q) {
  q[0] = 0.5f * c + 0.5f * d;
  q[1] = -0.5f * b + 1.5f * c;
  q[2] = (1.0f / 3.0f) * c + (5.0f / 6.0f) * d - (1.0f / 6.0f) * e;
  q[3] = (1.0f / 3.0f) * a - (7.0f / 6.0f) * b + (11.0f / 6.0f) * c;
}

// One side of a sample: qhat = sum_k softmax(z)_k c_k, q = sum_k y_k c_k with
// c_k the candidates on the side's normalised stencil x (x0..x4 on the left,
// the mirror x5..x1 on the right); r = (qhat - q) / kValueScale, whose square
// is the side's loss, and dz the gradient of the loss to its logits, scaled
// by 1/n.  Returns |qhat - q|.
__device__ __forceinline__ float side_loss(const float* z, const float* y, const float* x,
                                           float inv_n, float& r, float* dz) {
  float cand[4];
  candidates(x[0], x[1], x[2], x[3], x[4], cand);
  float m = z[0];
#pragma unroll
  for (int k = 1; k < 4; k++) m = fmaxf(m, z[k]);
  float e[4], s = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    e[k] = __expf(z[k] - m);
    s += e[k];
  }
  float qh = 0.0f, qt = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    e[k] = e[k] / s;
    qh += e[k] * cand[k];
    qt += y[k] * cand[k];
  }
  r = (qh - qt) * (1.0f / kValueScale);
  const float g = 2.0f * r * (1.0f / kValueScale) * inv_n;
#pragma unroll
  for (int k = 0; k < 4; k++) dz[k] = g * e[k] * (cand[k] - qh);
  return fabsf(qh - qt);
}

// One wave's exchange between the layers and the weight gradients, rows of 32
// samples (a row's stride spreads 32 rows over all banks, for 4 bf16 and for
// 4 floats a lane): activations and the gradient of one layer at a time.
constexpr int kSampleRow = 36;
struct alignas(16) GradTile {
  uint16_t h1[MLP_H * kSampleRow], h2[MLP_H * kSampleRow], x[MLP_NI * kSampleRow];
  float d[MLP_H * kSampleRow];
};

// Orders a wave's own LDS writes and reads for the compiler (the hardware
// runs them in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Four floats from any address of a float.
struct __attribute__((packed, aligned(4))) Float4u {
  float v[4];
};
__device__ __forceinline__ bf16x4 load_bf16x4(const float* p) {
  const Float4u f = *reinterpret_cast<const Float4u*>(p);
  return pack_bf16x4(f.v[0], f.v[1], f.v[2], f.v[3]);
}

// G += d a^T over the tile's samples (d: rows of T.d below `rows`, zero above;
// a: rows of `act` below `arows`), and the sum of d's row l % 32 over the
// samples (the bias gradient) as the return value.
__device__ __forceinline__ float grad_outer(const GradTile& T, const uint16_t* act, int rows,
                                            int arows, f32x16& G) {
  const int l = threadIdx.x & 63, i = l & 31, kh = (l >> 5) * 4;
  float sum = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    float4 d = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    bf16x4 a = {0, 0, 0, 0};
    if (i < rows) d = *reinterpret_cast<const float4*>(&T.d[i * kSampleRow + 8 * q + kh]);
    if (i < arows) a = *reinterpret_cast<const bf16x4*>(&act[i * kSampleRow + 8 * q + kh]);
    sum = ((sum + d.x) + d.y + d.z) + d.w;
    G = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(pack_bf16x4(d.x, d.y, d.z, d.w), a, G, 0, 0, 0);
  }
  return sum + __shfl_xor(sum, 32);
}

// Forward + backward over n samples; each workgroup writes its partial
// gradient (and loss) to part[blockIdx.x][MLP_NPARAM + 1].
//
// A wave has one tile of 32 samples at 65 536 samples, so the kernel is one
// tile's chain of seven products long, with the exchange between them.  The
// layers run transposed, h^T = W x^T (see the inference in mlp.hpp): a
// layer's accumulators are the next product's operand in both directions, the
// weights come straight from the parameters (rows as 4 floats a lane, columns
// coalesced), and each half of the wave forms one side of the sample's loss.
// Only the weight gradients, whose contraction is over the samples, go
// through LDS, with 8- and 16-byte reads free of bank conflicts.  Before, all
// operands were 2-byte LDS reads of rows 64 bytes apart (8 lanes a bank) and
// half the lanes idled in the loss: 24 us at 65 536 samples; now 15.2 us with
// 4 waves a workgroup and 10.3 us with 8 (half the partial rows to write).
// Masters, biases, loss, gradients and every sum are float; operands of the
// products are rounded to bf16.
//
// The loss of a sample: the squares of side_loss's two r, and binary
// cross-entropy of the confidence logit against c; c < 0 asks for the label
// to be formed here: 1 when both |qhat - q| < kConfTol, else 0.
__global__ __launch_bounds__(64 * GRAD_WAVES) void mlp_grad_kernel(
    const float* __restrict__ P, const float* __restrict__ X, const float* __restrict__ Y,
    const float* __restrict__ Cc, int64_t n, float* __restrict__ part) {
  // after its last tile a wave's results take the place of its tile
  __shared__ GradTile tiles[GRAD_WAVES];
  static_assert(sizeof(GradTile) >= sizeof(float) * (MLP_NPARAM + 1), "results fit the tile");
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int i = l & 31, half = l >> 5, kh = half * 4;
  GradTile& T = tiles[wave];
  const float inv_n = 1.0f / (float)n;
  // operands of the forward products (rows of W) and of the backward ones
  // (columns), and the biases of the lane's accumulator rows
  bf16x4 w1 = load_bf16x4(P + P_W1 + i * MLP_NI + kh), w2[4], w3[4], w2t[4], w3t[2];
  float b1[16], b2[16], b3[4];
#pragma unroll
  for (int q = 0; q < 4; q++) {
    w2[q] = load_bf16x4(P + P_W2 + i * MLP_H + 8 * q + kh);
    w3[q] = bf16x4{0, 0, 0, 0};
    if (i < MLP_NO) w3[q] = load_bf16x4(P + P_W3 + i * MLP_H + 8 * q + kh);
    const float* c2 = P + P_W2 + (8 * q + kh) * MLP_H + i;
    w2t[q] = pack_bf16x4(c2[0], c2[MLP_H], c2[2 * MLP_H], c2[3 * MLP_H]);
#pragma unroll
    for (int t = 0; t < 4; t++) {
      b1[4 * q + t] = P[P_B1 + 8 * q + kh + t];
      b2[4 * q + t] = P[P_B2 + 8 * q + kh + t];
    }
    b3[q] = P[P_B3 + kh + q];
  }
  const float* c3 = P + P_W3 + kh * MLP_H + i;
  w3t[0] = pack_bf16x4(c3[0], c3[MLP_H], c3[2 * MLP_H], c3[3 * MLP_H]);
  w3t[1] = pack_bf16x4(half == 0 ? P[P_W3 + 8 * MLP_H + i] : 0.0f, 0.0f, 0.0f, 0.0f);
  const float b3c = P[P_B3 + 8];

  f32x16 g1 = zero16(), g2 = zero16(), g3 = zero16();
  float gb1 = 0.0f, gb2 = 0.0f, gb3 = 0.0f, loss = 0.0f;
  const int64_t ntile = (n + 31) / 32;
  for (int64_t t0 = (int64_t)blockIdx.x * GRAD_WAVES + wave; t0 < ntile;
       t0 += (int64_t)gridDim.x * GRAD_WAVES) {
    const int64_t s = t0 * 32 + i;
    const bool valid = s < n;
    Float4u xl = {}, xr = {}, y = {};
    float c = 0.0f;
    if (valid) {
      xl = *reinterpret_cast<const Float4u*>(X + s * MLP_NI);
      xr = *reinterpret_cast<const Float4u*>(X + s * MLP_NI + 4);
      y = *reinterpret_cast<const Float4u*>(Y + s * 8 + kh);
      c = Cc ? Cc[s] : -1.0f;
    }
    // forward; the lane's rows of each layer are 8 q + kh + t, its column
    // sample i
    const bf16x4 xb = half ? pack_bf16x4(xr.v[0], xr.v[1], xr.v[2], xr.v[3])
                           : pack_bf16x4(xl.v[0], xl.v[1], xl.v[2], xl.v[3]);
#pragma unroll
    for (int t = 0; t < 4; t++) T.x[(kh + t) * kSampleRow + i] = (uint16_t)xb[t];
    auto activate = [&](const f32x16& acc, const float* b, uint16_t* row, bf16x4* h) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
          v[t] = acc[4 * q + t] + b[4 * q + t];
          v[t] = v[t] > 0.0f ? v[t] : 0.0f;
        }
        h[q] = pack_bf16x4(v[0], v[1], v[2], v[3]);
#pragma unroll
        for (int t = 0; t < 4; t++) row[(8 * q + kh + t) * kSampleRow + i] = (uint16_t)h[q][t];
      }
    };
    bf16x4 h1[4], h2[4];
    f32x16 acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w1, xb, zero16(), 0, 0, 0);
    activate(acc, b1, T.h1, h1);
    acc = zero16();
#pragma unroll
    for (int q = 0; q < 4; q++)
      acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w2[q], h1[q], acc, 0, 0, 0);
    activate(acc, b2, T.h2, h2);
    acc = zero16();
#pragma unroll
    for (int q = 0; q < 4; q++)
      acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w3[q], h2[q], acc, 0, 0, 0);
    // loss and dz: lane l holds the logits of side l / 32 of sample i, and the
    // lower half the confidence's
    float z[4], dz[4], r;
#pragma unroll
    for (int k = 0; k < 4; k++) z[k] = acc[k] + b3[k];
    const float xs[5] = {half ? xr.v[1] : xl.v[0], half ? xr.v[0] : xl.v[1],
                         half ? xl.v[3] : xl.v[2], half ? xl.v[2] : xl.v[3],
                         half ? xl.v[1] : xr.v[0]};
    float err = side_loss(z, y.v, xs, inv_n, r, dz);
    err = fmaxf(err, __shfl_xor(err, 32));
    if (c < 0.0f) c = err < kConfTol ? 1.0f : 0.0f;
    const float zc = acc[4] + b3c;
    float dc = (1.0f / (1.0f + __expf(-zc)) - c) * inv_n, ls = r * r;
    if (half) dc = 0.0f;
    else ls += fmaxf(zc, 0.0f) - zc * c + log1pf(__expf(-fabsf(zc)));
    if (valid) {
      loss += ls * inv_n;
    } else {
      dc = 0.0f;
#pragma unroll
      for (int k = 0; k < 4; k++) dz[k] = 0.0f;
    }
    const bf16x4 dz0 = pack_bf16x4(dz[0], dz[1], dz[2], dz[3]);
    const bf16x4 dz1 = pack_bf16x4(dc, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int t = 0; t < 4; t++) {
      T.d[(kh + t) * kSampleRow + i] = dz[t];
      T.d[(8 + kh + t) * kSampleRow + i] = t == 0 ? dc : 0.0f;
    }
    wave_lds_fence();
    // gW3[j][k] += sum_s dz[s][j] h2[s][k], gb3[j] += sum_s dz[s][j]
    gb3 += grad_outer(T, T.h2, 16, MLP_H, g3);
    wave_lds_fence();
    // d[k][s] = (sum_j W[j][k] d'[j][s]) * relu'(h)
    auto through_relu = [&](const f32x16& v, const bf16x4* h, bf16x4* d) {
#pragma unroll
      for (int q = 0; q < 4; q++) {
        float m[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
          m[t] = bf2f((uint16_t)h[q][t]) > 0.0f ? v[4 * q + t] : 0.0f;
          T.d[(8 * q + kh + t) * kSampleRow + i] = m[t];
        }
        d[q] = pack_bf16x4(m[0], m[1], m[2], m[3]);
      }
    };
    bf16x4 d[4];
    acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w3t[0], dz0, zero16(), 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w3t[1], dz1, acc, 0, 0, 0);
    through_relu(acc, h2, d);
    wave_lds_fence();
    // gW2[j][k] += sum_s dh2[s][j] h1[s][k]
    gb2 += grad_outer(T, T.h1, MLP_H, MLP_H, g2);
    wave_lds_fence();
    acc = zero16();
#pragma unroll
    for (int q = 0; q < 4; q++)
      acc = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(w2t[q], d[q], acc, 0, 0, 0);
    through_relu(acc, h1, d);
    wave_lds_fence();
    // gW1[j][k] += sum_s dh1[s][j] x[s][k]
    gb1 += grad_outer(T, T.x, MLP_H, MLP_NI, g1);
    wave_lds_fence();
  }
  float* R = reinterpret_cast<float*>(&T);
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const int i = mrow(l, r), k = mcol(l);
    if (k < MLP_NI) R[P_W1 + i * MLP_NI + k] = g1[r];
    R[P_W2 + i * MLP_H + k] = g2[r];
    if (i < MLP_NO) R[P_W3 + i * MLP_H + k] = g3[r];
  }
  if (l < 32) {
    R[P_B1 + l] = gb1;
    R[P_B2 + l] = gb2;
  }
  if (l < MLP_NO) R[P_B3 + l] = gb3;
  // wave loss: sum over lanes
  float ls = loss;
  for (int o = 32; o > 0; o >>= 1) ls += __shfl_xor(ls, o);
  if (l == 0) R[MLP_NPARAM] = ls;
  __syncthreads();
  for (int e = tid; e < MLP_NPARAM + 1; e += blockDim.x) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < GRAD_WAVES; w++) s += reinterpret_cast<const float*>(&tiles[w])[e];
    part[(int64_t)blockIdx.x * (MLP_NPARAM + 1) + e] = s;
  }
}

// Fixed-order sum of the workgroup partials (nblk rows of MLP_NPARAM + 1).
// A workgroup sums kRedCols columns: kRedRows row classes (rows r, r +
// kRedRows, ...) side by side, then the classes in order.  The reads are the
// whole cost (1.7 MB: 256 rows at 65 536 samples); one lane per column, each
// walking all rows, left 7 workgroups with one load in flight per lane: 119
// us at 512 rows.  This split has 52 workgroups of 16 waves, each lane with
// four loads in flight: 7.2 us at 512 rows, 4.7 us at 256.
constexpr int kRedCols = 32, kRedRows = 32;
__global__ __launch_bounds__(kRedCols * kRedRows) void mlp_reduce_kernel(const float* part,
                                                                         int nblk, float* grad,
                                                                         float* loss) {
  constexpr int UNR = 4, W = MLP_NPARAM + 1;
  __shared__ float acc[kRedRows][kRedCols];
  const int col = threadIdx.x % kRedCols, r = threadIdx.x / kRedCols;
  const int e = blockIdx.x * kRedCols + col;
  float s[UNR] = {};
  if (e < W) {
    for (int b = r; b < nblk; b += kRedRows * UNR) {
#pragma unroll
      for (int k = 0; k < UNR; k++)
        if (b + k * kRedRows < nblk) s[k] += part[(int64_t)(b + k * kRedRows) * W + e];
    }
  }
  acc[r][col] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  for (int h = kRedRows / 2; h > 0; h /= 2) {
    if (r < h) acc[r][col] += acc[r + h][col];
    __syncthreads();
  }
  if (r != 0 || e >= W) return;
  if (e < MLP_NPARAM)
    grad[e] = acc[0][col];
  else
    *loss = acc[0][col];
}

// The network as the stage kernel evaluates it (packed bf16 parameters,
// activations in registers, 64 samples per wave): one sample per lane,
// lanes past n evaluate zeros and store nothing.
__global__ __launch_bounds__(256) void mlp_infer_kernel(const uint16_t* packed, const float* X,
                                                       int64_t n, float* out) {
  __shared__ MlpLds W;
  __shared__ MlpBiasLds B;
  const int tid = threadIdx.x;
  mlp_stage_bf16(W, packed, tid, 256);
  __syncthreads();
  mlp_bias_stage(B, W, tid, 256);
  MlpRegs R;
  mlp_regs_load(W, R);
  __syncthreads();
  const int64_t s = (int64_t)blockIdx.x * 256 + tid;
  float x[MLP_NI], z[MLP_NO];
#pragma unroll
  for (int k = 0; k < MLP_NI; k++) x[k] = s < n ? X[s * MLP_NI + k] : 0.0f;
  mlp_logits_wave(x, R, B, z);
  if (s < n) {
#pragma unroll
    for (int k = 0; k < MLP_NO; k++) out[s * MLP_NO + k] = z[k];
  }
}

__global__ __launch_bounds__(64 * MLP_WAVES) void mlp_forward_kernel(const float* P,
                                                                     const float* X, int64_t n,
                                                                     float* out) {
  __shared__ MlpLds W;
  __shared__ MlpTile tiles[MLP_WAVES];
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  mlp_stage_f32(W, P, tid, blockDim.x);
  __syncthreads();
  MlpTile& T = tiles[wave];
  const int64_t ntile = (n + 31) / 32;
  for (int64_t t = (int64_t)blockIdx.x * MLP_WAVES + wave; t < ntile;
       t += (int64_t)gridDim.x * MLP_WAVES) {
    const int64_t s0 = t * 32;
    for (int e = l; e < 32 * MLP_NI; e += 64) {
      const int64_t s = s0 + e / MLP_NI;
      T.x[e] = f2bf(s < n ? X[s * MLP_NI + e % MLP_NI] : 0.0f);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    mlp_tile_forward(W, T);
    for (int e = l; e < 32 * MLP_NO; e += 64) {
      const int64_t s = s0 + e / MLP_NO;
      if (s < n) out[s * MLP_NO + e % MLP_NO] = T.z[(e / MLP_NO) * 16 + e % MLP_NO];
    }
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
  }
}

__global__ void mlp_adam_kernel(float* P, const float* G, float* M, float* V, float lr, float b1,
                                float b2, float eps, float c1, float c2) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= MLP_NPARAM) return;
  const float g = G[e];
  const float m = b1 * M[e] + (1.0f - b1) * g;
  const float v = b2 * V[e] + (1.0f - b2) * g * g;
  M[e] = m;
  V[e] = v;
  P[e] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
}

__global__ void mlp_pack_kernel(const float* P, uint16_t* out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < MLP_NPARAM) out[e] = f2bf(P[e]);
}

// Training samples: for every face of every axis and every characteristic
// field, the network inputs and the eq. (28) weights of both sides (FP64,
// read straight from global memory; this is data preparation, not the hot
// path).  Face-field g (axis-major, then face, then field) is taken when
// g % stride == 0 and written at row g / stride < max.
template <int NDIM>
__global__ void mlp_samples_kernel(const double* U, int64_t n0, int64_t n1, int64_t n2, int bclo0,
                                   int bchi0, int bclo1, int bchi1, int bclo2, int bchi2,
                                   double eps, int64_t stride, int64_t maxs, float* X, float* Y) {
  constexpr int NC = 4 + NDIM, NT = NDIM - 1;
  const int64_t n[3] = {n0, n1, n2};
  const int bl[3] = {bclo0, bclo1, bclo2}, bh[3] = {bchi0, bchi1, bchi2};
  const int64_t N = n0 * n1 * n2;
  int64_t base = 0;
  for (int D = 0; D < NDIM; D++) {
    const int64_t nf = N / n[D] * (n[D] + 1);
    for (int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; f < nf;
         f += (int64_t)gridDim.x * blockDim.x) {
      const int64_t g0 = (base + f) * NC;
      // any of this face's fields selected?
      const int64_t first = ((g0 + stride - 1) / stride) * stride;
      if (first >= g0 + NC || first / stride >= maxs) continue;
      // face f: index along D and the line it sits on
      const int64_t fl = f % (n[D] + 1), line = f / (n[D] + 1);
      int64_t sL = 1, sA = 0, sT = 0, a = 0, tt = 0;
      if (D == 0) {
        sL = 1; a = line; sA = n0;
      } else if (D == 1) {
        sL = n0; a = line % n0; sA = 1; tt = line / n0; sT = n0 * n1;
      } else {
        sL = n0 * n1; a = line % n0; sA = 1; tt = line / n0; sT = n0;
      }
      double q[6][NC];
      for (int j = 0; j < 6; j++) {
        bool flip;
        const int64_t li = bc_index(fl - 3 + j, n[D], bl[D], bh[D], flip);
        cell_prim<NDIM>(U, N, a * sA + li * sL + tt * sT, q[j]);
        if (flip) q[j][1 + D] = -q[j][1 + D];
      }
      const double rb = 0.5 * (q[2][0] + q[3][0]), pb = 0.5 * (q[2][1 + NDIM] + q[3][1 + NDIM]);
      const double Gb = 0.5 * (q[2][2 + NDIM] + q[3][2 + NDIM]);
      const double Pb = 0.5 * (q[2][3 + NDIM] + q[3][3 + NDIM]);
      const double c2 = sound2<double>(rb, pb, Gb, Pb), c = sqrt(c2);
      const double aa = rb * c / 2.0, b = 1.0 / c2;
      for (int m = 0; m < NC; m++) {
        const int64_t g = g0 + m;
        if (g % stride || g / stride >= maxs) continue;
        double w[6];
        for (int j = 0; j < 6; j++) {
          if (m == 0) w[j] = (-aa) * q[j][1 + D] + 0.5 * q[j][1 + NDIM];
          else if (m == NC - 1) w[j] = aa * q[j][1 + D] + 0.5 * q[j][1 + NDIM];
          else if (m == 1) w[j] = q[j][0] - b * q[j][1 + NDIM];
          else if (m < 2 + NT) w[j] = q[j][1 + ((m - 2) < D ? (m - 2) : (m - 1))];
          else if (m == 2 + NT) w[j] = q[j][2 + NDIM];
          else w[j] = q[j][3 + NDIM];
        }
        const int64_t row = g / stride;
        float x[8], f6, f7;
        mlp_material(Gb, Pb, f6, f7);
        mlp_features<double>(w, f6, f7, x);
        for (int k = 0; k < 8; k++) X[row * 8 + k] = x[k];
        for (int side = 0; side < 2; side++) {
          double v[5];
          for (int k = 0; k < 5; k++) v[k] = side ? w[5 - k] : w[k];
          const Ind<double> s = indicators<double>(v[0], v[1], v[2], v[3], v[4]);
          const Alpha al = alphas_f64(s, W_MODIFIED, eps, false);
          const double sum = ((al.a1 + al.a2) + al.a3) + al.a4;
          Y[row * 8 + 4 * side + 0] = float(al.a1 / sum);
          Y[row * 8 + 4 * side + 1] = float(al.a2 / sum);
          Y[row * 8 + 4 * side + 2] = float(al.a3 / sum);
          Y[row * 8 + 4 * side + 3] = float(al.a4 / sum);
        }
      }
    }
    base += nf;
  }
}

}  // namespace isw

namespace {
int mlp_blocks(int64_t n, int waves) {
  int64_t b = (n + 32 * waves - 1) / (32 * waves);
  if (b > 1024) b = 1024;
  if (b < 1) b = 1;
  return (int)b;
}
}  // namespace

extern "C" {

int isweno_mlp_samples(isweno_ctx* ctx, const isweno_grid* g, const isweno_opts* o, const double* U,
                       float* X, float* Y, int64_t max_samples, int64_t stride, int64_t* count,
                       void* stream) {
  if (!ctx || !g || !o || !U || !X || !Y || !count || max_samples < 1 || stride < 1)
    return ISWENO_ERR_ARG;
  int r;
  // the same grid and option checks as the solver: the sampler stages the
  // same ghost cells (a reflective end needs at least 3 cells)
  if ((r = isw::check_grid(g)) != ISWENO_OK) return r;
  if ((r = isw::check_opts(o)) != ISWENO_OK) return r;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int64_t N = g->n[0] * g->n[1] * g->n[2];
  int64_t total = 0;
  for (int d = 0; d < g->ndim; d++) total += N / g->n[d] * (g->n[d] + 1) * (4 + g->ndim);
  const int64_t rows = (total + stride - 1) / stride;
  const int64_t written = rows < max_samples ? rows : max_samples;
  const dim3 grid(1024), block(256);
  if (g->ndim == 1)
    hipLaunchKernelGGL(isw::mlp_samples_kernel<1>, grid, block, 0, s, U, g->n[0], g->n[1], g->n[2],
                       g->bc_lo[0], g->bc_hi[0], g->bc_lo[1], g->bc_hi[1], g->bc_lo[2],
                       g->bc_hi[2], o->eps, stride, max_samples, X, Y);
  else if (g->ndim == 2)
    hipLaunchKernelGGL(isw::mlp_samples_kernel<2>, grid, block, 0, s, U, g->n[0], g->n[1], g->n[2],
                       g->bc_lo[0], g->bc_hi[0], g->bc_lo[1], g->bc_hi[1], g->bc_lo[2],
                       g->bc_hi[2], o->eps, stride, max_samples, X, Y);
  else
    hipLaunchKernelGGL(isw::mlp_samples_kernel<3>, grid, block, 0, s, U, g->n[0], g->n[1], g->n[2],
                       g->bc_lo[0], g->bc_hi[0], g->bc_lo[1], g->bc_hi[1], g->bc_lo[2],
                       g->bc_hi[2], o->eps, stride, max_samples, X, Y);
  if (hipGetLastError() != hipSuccess) return ISWENO_ERR_DEVICE;
  if (hipMemcpyAsync(count, &written, sizeof(int64_t), hipMemcpyHostToDevice, s) != hipSuccess)
    return ISWENO_ERR_DEVICE;
  return hipStreamSynchronize(s) == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

int isweno_mlp_infer(isweno_ctx* ctx, const uint16_t* packed, const float* X, int64_t n,
                     float* out, void* stream) {
  if (!ctx || !packed || !X || !out || n < 0) return ISWENO_ERR_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  if (n == 0) return ISWENO_OK;
  const int64_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffffLL) return ISWENO_ERR_ARG;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(isw::mlp_infer_kernel, dim3((unsigned)blocks), dim3(256), 0, s, packed, X, n,
                     out);
  return hipGetLastError() == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

int isweno_mlp_forward(isweno_ctx* ctx, const float* P, const float* X, int64_t n, float* out,
                       void* stream) {
  if (!ctx || !P || !X || !out || n < 0) return ISWENO_ERR_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  if (n == 0) return ISWENO_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(isw::mlp_forward_kernel, dim3(mlp_blocks(n, isw::MLP_WAVES)),
                     dim3(64 * isw::MLP_WAVES), 0, s, P, X, n, out);
  return hipGetLastError() == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

int isweno_mlp_loss_grad(isweno_ctx* ctx, const float* P, const float* X, const float* Y,
                         const float* Cc, int64_t n, float* loss, float* grad, void* stream) {
  if (!ctx || !P || !X || !Y || !loss || !grad || n < 1) return ISWENO_ERR_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int nb = mlp_blocks(n, isw::GRAD_WAVES);
  // partial gradients in the context's own buffer (grown on demand; calls
  // on one context do not overlap, see isweno.h)
  if (nb > ctx->mlp_part_blocks) {
    if (ctx->mlp_part) {
      if (hipDeviceSynchronize() != hipSuccess) return ISWENO_ERR_DEVICE;
      (void)hipFree(ctx->mlp_part);
      ctx->mlp_part = nullptr;
      ctx->mlp_part_blocks = 0;
    }
    if (hipMalloc(&ctx->mlp_part, sizeof(float) * (size_t)nb * (isw::MLP_NPARAM + 1)) !=
        hipSuccess)
      return ISWENO_ERR_DEVICE;
    ctx->mlp_part_blocks = nb;
  }
  hipLaunchKernelGGL(isw::mlp_grad_kernel, dim3(nb), dim3(64 * isw::GRAD_WAVES), 0, s, P, X, Y, Cc,
                     n, ctx->mlp_part);
  if (hipGetLastError() != hipSuccess) return ISWENO_ERR_DEVICE;
  hipLaunchKernelGGL(isw::mlp_reduce_kernel,
                     dim3((isw::MLP_NPARAM + isw::kRedCols) / isw::kRedCols),
                     dim3(isw::kRedCols * isw::kRedRows), 0, s, ctx->mlp_part, nb, grad, loss);
  return hipGetLastError() == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

int isweno_mlp_adam(isweno_ctx* ctx, float* P, const float* G, float* M, float* V, int32_t step,
                    float lr, float beta1, float beta2, float eps, void* stream) {
  if (!ctx || !P || !G || !M || !V || step < 1) return ISWENO_ERR_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
  hipLaunchKernelGGL(isw::mlp_adam_kernel, dim3((isw::MLP_NPARAM + 255) / 256), dim3(256), 0, s, P,
                     G, M, V, lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

int isweno_mlp_pack(isweno_ctx* ctx, const float* P, uint16_t* packed, void* stream) {
  if (!ctx || !P || !packed) return ISWENO_ERR_ARG;
  if (hipSetDevice(ctx->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(isw::mlp_pack_kernel, dim3((isw::MLP_NPARAM + 255) / 256), dim3(256), 0, s, P,
                     packed);
  return hipGetLastError() == hipSuccess ? ISWENO_OK : ISWENO_ERR_DEVICE;
}

}  // extern "C"
