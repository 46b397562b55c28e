// Surrogate for the inverse internal equation of state theta(eps).
//
// Network: x = (ln eps - in_c)/in_s, h1 = tanh(W1 x + b1), h2 = tanh(W2 h1 + b2),
// y = W3 . h2 + b3, theta = exp(out_c + out_s y); 32 hidden units per layer,
// weights packed W1[32] b1[32] W2[32][32] b2[32] W3[32] b3 (1153 values).
//
// Inference: the 32x32 layer runs on the matrix cores in BF16 with FP32
// accumulation (the input and output layers, on the vector units, use the
// FP32 weights) as H2^T = W2 H1^T with one v_mfma_f32_32x32x16_bf16 per
// (32 particles x 16 inputs) block: the weights are the A operand (constant),
// each lane builds its B-operand column of tanh(W1 x + b1) for the particle it
// serves, and the accumulator leaves every lane with 16 hidden units of one
// particle, so the output layer is a 16-term dot product plus one cross-half
// shuffle.
//
// Training runs in FP32 on the GPU: forward and backward of 16 samples per wave
// with the 32x32 products on the matrix cores in FP32, per-block gradient sums
// in a fixed order, a second kernel adds the block partials in block order and
// applies Adam.  Samples
// are theta log-uniform in the training range, eps = eps(theta) from the EOS.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "common.h"
#include "eos.h"

namespace dpde {

constexpr int kH = 32;
constexpr int kNParam = kH + kH + kH * kH + kH + kH + 1;  // 1153
constexpr int OFF_W1 = 0, OFF_B1 = kH, OFF_W2 = 2 * kH, OFF_B2 = OFF_W2 + kH * kH;
constexpr int OFF_W3 = OFF_B2 + kH, OFF_B3 = OFF_W3 + kH;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct MlpState {
  bool trained = false;
  float* w = nullptr;       // FP32 master weights
  uint16_t* wb = nullptr;   // BF16 bit patterns used by inference
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  float* gpart = nullptr;   // per-block gradient partials
  double* lpart = nullptr;  // per-block loss partials
  float* loss = nullptr;    // loss per iteration
  float* gsum = nullptr;    // summed gradient (gradient checks)
  float* xs = nullptr;      // training inputs
  float* ts = nullptr;      // training targets
  int64_t nsamp = 0;
  int64_t loss_cap = 0;
  int gblocks = 0;
  double norm[4] = {0, 1, 0, 1};  // in_c, in_s, out_c, out_s
  double eps_lo = 0, eps_hi = 0;
  std::vector<void*> allocs;
};

// ---- conversions ----------------------------------------------------------------
__host__ __device__ inline uint16_t f32_to_bf16_bits(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even (finite inputs)
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __uint_as_float((uint32_t)b << 16);
}

__device__ __forceinline__ float fast_tanh(float x) {
  // tanh x = 1 - 2/(e^{2x} + 1); e^{2x} = 2^{2x log2 e}
  const float e = __builtin_amdgcn_exp2f(2.8853900817779268f * x);
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// ---- inference: every lane of the wave must call; returns this lane's y ---------
// The 32x32 layer is the matrix-core product: W2 and the hidden activations
// enter it in BF16.  The input and output layers (vectors, evaluated on the
// vector units) keep the FP32 master weights.
// 32 particles: lane l serves particle l % 32 (both half-waves pass that
// particle's x) and every lane gets that particle's y.
__device__ __forceinline__ float mlp_wave32(const float* __restrict__ wf,
                                            const uint16_t* __restrict__ wb, float xp) {
  const int l = threadIdx.x % kWave;
  const int half = l >> 5, col = l & 31;
  bf16x8 a[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      a[ks][e] = __builtin_bit_cast(__bf16, wb[OFF_W2 + col * kH + ks * 16 + 8 * half + e]);
  f32x16 acc = {};
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    bf16x8 b;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = ks * 16 + 8 * half + e;
      const float h = fast_tanh(wf[OFF_W1 + k] * xp + wf[OFF_B1 + k]);
      b[e] = __builtin_bit_cast(__bf16, f32_to_bf16_bits(h));
    }
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], b, acc, 0, 0, 0);
  }
  float s = 0.0f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int u = 8 * (r >> 2) + 4 * half + (r & 3);
    s += wf[OFF_W3 + u] * fast_tanh(acc[r] + wf[OFF_B2 + u]);
  }
  s += __shfl_xor(s, 32, kWave);
  return s + wf[OFF_B3];
}

// 64 particles: lane l passes the x of particle l and gets its y.
__device__ __forceinline__ float mlp_wave(const float* __restrict__ wf,
                                          const uint16_t* __restrict__ wb, float x) {
  const int l = threadIdx.x % kWave;
  const int half = l >> 5, col = l & 31;
  float y[2];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) y[mb] = mlp_wave32(wf, wb, __shfl(x, 32 * mb + col, kWave));
  return half ? y[1] : y[0];
}

struct MlpDev {
  const float* wf;     // FP32 master weights (input and output layers)
  const uint16_t* wb;  // BF16 copy (the matrix-core layer W2)
  double in_c, in_s, out_c, out_s, eps_lo, eps_hi;
};

// theta (OUT_INV = 0) or 1/theta (OUT_INV = 1) for n energies.  mode 1: the
// network inside [eps_lo, eps_hi], Newton outside; mode 2: Newton started
// from the network's estimate (or the asymptote outside the range); mode 0:
// Newton alone.  No lane leaves before the matrix-core step.
// Network input for eps: normalised log, clamped to the training interval.
__device__ __forceinline__ float mlp_input(const MlpDev& m, double e) {
  double xd = (log(e > 0.0 ? e : 1.0) - m.in_c) / m.in_s;
  xd = xd < -1.0 ? -1.0 : (xd > 1.0 ? 1.0 : xd);
  return (float)xd;
}

// theta from the network output y (modes 1, 2) or by Newton (mode 0, and
// outside the training range in mode 1).
__device__ __forceinline__ double theta_from_net(const Phys& P, const MlpDev& m, int mode,
                                                 double e, float y, int& it) {
  it = 0;
  if (P.eos == 0) return e / P.cv;
  const bool in_range = e >= m.eps_lo && e <= m.eps_hi;
  const double th_net = mode != 0 ? exp(m.out_c + m.out_s * (double)y) : 0.0;
  if (mode == 1 && in_range) return th_net;
  return theta_newton_dev(P, e, (mode == 2 && in_range) ? th_net : theta_start_dev(P, e), it);
}

template <int OUT_INV>
__global__ __launch_bounds__(256) void k_theta(const double* __restrict__ eps, double* __restrict__ out,
                                               int64_t ostride, int32_t* __restrict__ iters,
                                               int64_t n, Phys P, MlpDev m, int mode,
                                               uint32_t* status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = i < n;
  const double e = valid ? eps[i] : 1.0;
  float y = 0.0f;
  if (P.eos != 0 && mode != 0) y = mlp_wave(m.wf, m.wb, mlp_input(m, e));  // uniform
  int it;
  const double th = theta_from_net(P, m, mode, e, y, it);
  if (!valid) return;
  if (!(e > 0.0)) {
    if (status) atomicOr(status, ST_NEG_EINT);
    return;
  }
  if (!(th > 0.0) || !isfinite(th)) {
    if (status) atomicOr(status, ST_EOS);
  }
  out[i * ostride] = OUT_INV ? 1.0 / th : th;
  if (iters) iters[i] = it;
}

__global__ void k_eos_energy(const double* __restrict__ theta, double* __restrict__ eps, int64_t n,
                             Phys P) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) eps[i] = eos_energy_dev(P, theta[i]);
}

// y for normalised inputs (test hook for the inference path).
__global__ __launch_bounds__(256) void k_mlp_eval(const float* __restrict__ wf,
                                                  const uint16_t* __restrict__ wb,
                                                  const float* __restrict__ x, float* __restrict__ y,
                                                  int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const float xi = i < n ? x[i] : 0.0f;
  const float v = mlp_wave(wf, wb, xi);
  if (i < n) y[i] = v;
}

// ---- training ---------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTrainThreads = 256;
constexpr int kTrainWaves = kTrainThreads / kWave;
constexpr int kTrainCols = 16;     // samples a wave takes at once: the columns of its products
constexpr int kTrainBlocks = 64;   // most blocks, and so partial gradients, of one batch
constexpr int kLd = kH + 1;        // padded LDS row

// Blocks for a batch of n samples: each of a block's four waves takes 16.
inline int train_blocks(int64_t n) {
  const int64_t per = kTrainWaves * kTrainCols;
  return (int)std::min<int64_t>(kTrainBlocks, (n + per - 1) / per);
}

// Training samples: theta log-uniform in [lo, hi] from Philox words keyed by
// the seed (counter = sample index), eps = eps(theta).
__global__ void k_mlp_samples(uint64_t seed, int64_t n, double lnlo, double lnhi, Phys P,
                              double in_c, double in_s, double out_c, double out_s,
                              float* __restrict__ xs, float* __restrict__ ts) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  uint32_t w0 = (uint32_t)k, w1 = (uint32_t)(k >> 32), w2 = 0x534D504Cu, w3 = 0u;
  philox4x32_10<true>(w0, w1, w2, w3, (uint32_t)seed, (uint32_t)(seed >> 32));
  const double u = ((double)w0 + 0.5) * 2.3283064365386963e-10;
  const double lt = lnlo + u * (lnhi - lnlo);
  const double th = exp(lt);
  const double e = eos_energy_dev(P, th);
  xs[k] = (float)((log(e) - in_c) / in_s);
  ts[k] = (float)((lt - out_c) / out_s);
}

// Forward + backward of nb samples starting at sample `begin` (mod nsamp):
// block partial gradients of the mean squared error scaled by inv_batch.
//
// A batch is three 32 x 32 products per sample (W2 h1, W2^T d2 and the sum of
// d2 h1^T) between two layers of tanh, so at the usual 4096 samples the launch
// is bound by the length of one wave's chain, not by its arithmetic.  A wave
// therefore takes 16 samples, four lanes each, and the products run on the
// matrix cores in FP32 (v_mfma_f32_16x16x4_f32).  Sample c = lane % 16, group
// g = lane / 16; a lane holds the units u(q) = 16 (q / 4) + 4 g + q % 4 of its
// sample, q = 0..7.  That is the accumulator layout of the matrix instruction,
// and since the order of a product's inner index is free, the same registers
// are the B operand of the next product; only d2 and h1 go through LDS, for
// the product summed over samples.  Measured (batch 4096): 57.8 us with one
// thread per sample and the gradient summed from LDS by the vector units,
// 7.3 us in this form.
__global__ __launch_bounds__(kTrainThreads) void k_mlp_fwd_bwd(
    const float* __restrict__ w, const float* __restrict__ xs, const float* __restrict__ ts,
    int64_t nsamp, int64_t begin, int64_t nb, float inv_batch, float* __restrict__ gpart,
    double* __restrict__ lpart) {
  constexpr int kQ = kH / 4;            // units per lane
  constexpr int kRow = kWave + 1;       // padded row of the final sums
  constexpr int kT = kTrainCols * kLd;  // one wave's d2 or h1 by sample
  // the waves' transposed d2 and h1, then (after the samples) their sums
  __shared__ float buf[kTrainWaves * 4 * kQ * kRow];
  static_assert(2 * kT <= 4 * kQ * kRow && kH * kH <= 4 * kQ * kRow, "LDS regions");
  __shared__ double red[kTrainWaves];
  __shared__ float red3[kTrainWaves];
  const int tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const int c = lane % kTrainCols, g = lane / kTrainCols;
  auto unit = [g](int q) { return 16 * (q >> 2) + 4 * g + (q & 3); };
  float w1[kQ], b1[kQ], b2[kQ], w3[kQ];
  float wf[2][kQ], wt[2][kQ];  // W2 and its transpose as A operands
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    const int u = unit(q);
    w1[q] = w[OFF_W1 + u];
    b1[q] = w[OFF_B1 + u];
    b2[q] = w[OFF_B2 + u];
    w3[q] = w[OFF_W3 + u];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      wf[m][q] = w[OFF_W2 + (16 * m + c) * kH + u];
      wt[m][q] = w[OFF_W2 + u * kH + 16 * m + c];
    }
  }
  const float b3 = w[OFF_B3];
  f32x4 g2[2][2] = {};                // sum over samples of d2 h1^T, in tiles of 16 x 16
  float sw1[kQ], sb1[kQ], sb2[kQ], sw3[kQ], sb3 = 0.0f;
#pragma unroll
  for (int q = 0; q < kQ; ++q) sw1[q] = sb1[q] = sb2[q] = sw3[q] = 0.0f;
  double lsum = 0.0;
  float* td = buf + wv * 2 * kT;  // d2 by sample
  float* th = td + kT;            // h1 by sample
  const int64_t chunks = (nb + kTrainCols - 1) / kTrainCols;
  for (int64_t q0 = (int64_t)blockIdx.x * kTrainWaves + wv; q0 < chunks;
       q0 += (int64_t)gridDim.x * kTrainWaves) {  // uniform in the wave
    const int64_t s = q0 * kTrainCols + c;
    const bool live = s < nb;
    float x = 0.0f, t = 0.0f;
    if (live) {
      int64_t k = begin + s;
      if (k >= nsamp) k %= nsamp;
      x = xs[k];
      t = ts[k];
    }
    float h1[kQ], h2[kQ], d2[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) h1[q] = tanhf(w1[q] * x + b1[q]);
    float y = 0.0f;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      f32x4 z = {b2[4 * m], b2[4 * m + 1], b2[4 * m + 2], b2[4 * m + 3]};
#pragma unroll
      for (int q = 0; q < kQ; ++q) z = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[m][q], h1[q], z, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        h2[4 * m + r] = tanhf(z[r]);
        y += w3[4 * m + r] * h2[4 * m + r];
      }
    }
    y += __shfl_xor(y, 16, kWave);
    y += __shfl_xor(y, 32, kWave);
    const float err = live ? (y + b3) - t : 0.0f;
    if (g == 0) lsum += (double)err * (double)err;
    const float dy = 2.0f * err * inv_batch;
    sb3 += dy;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      // a lane beyond the batch adds nothing, whatever the weights are
      d2[q] = live ? dy * w3[q] * (1.0f - h2[q] * h2[q]) : 0.0f;
      sb2[q] += d2[q];
      sw3[q] += live ? dy * h2[q] : 0.0f;
      td[c * kLd + unit(q)] = d2[q];
      th[c * kLd + unit(q)] = live ? h1[q] : 0.0f;
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      f32x4 z = {};
#pragma unroll
      for (int q = 0; q < kQ; ++q) z = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[m][q], d2[q], z, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float h = h1[4 * m + r];
        const float d1 = live ? z[r] * (1.0f - h * h) : 0.0f;
        sb1[4 * m + r] += d1;
        sw1[4 * m + r] += d1 * x;
      }
    }
    // the wave's own LDS rows: a fence orders its writes and reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
    for (int k = 0; k < kTrainCols / 4; ++k) {
      const int row = (4 * k + g) * kLd + c;
      const float a0 = td[row], a1 = td[row + 16], h0 = th[row], hh = th[row + 16];
      g2[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, h0, g2[0][0], 0, 0, 0);
      g2[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, hh, g2[0][1], 0, 0, 0);
      g2[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, h0, g2[1][0], 0, 0, 0);
      g2[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, hh, g2[1][1], 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();  // the next samples overwrite the rows
  }
  // the block's sums, waves in order
  float* gp = gpart + (int64_t)blockIdx.x * kNParam;
  lsum = wave_sum(lsum);
#pragma unroll
  for (int off = kTrainCols / 2; off > 0; off >>= 1) sb3 += __shfl_xor(sb3, off, kWave);
  __syncthreads();
  if (lane == 0) {
    red[wv] = lsum;
    red3[wv] = sb3;
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        buf[wv * kH * kH + (16 * m + 4 * g + r) * kH + 16 * n + c] = g2[m][n][r];
  __syncthreads();
  for (int o = tid; o < kH * kH; o += kTrainThreads) {
    float v = 0.0f;
#pragma unroll
    for (int k = 0; k < kTrainWaves; ++k) v += buf[k * kH * kH + o];
    gp[OFF_W2 + o] = v;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kQ; ++q) {
    float* r0 = buf + (wv * 4 * kQ + q) * kRow + lane;
    r0[0] = sw1[q];
    r0[kQ * kRow] = sb1[q];
    r0[2 * kQ * kRow] = sb2[q];
    r0[3 * kQ * kRow] = sw3[q];
  }
  __syncthreads();
  {
    // value o / 2 of the 4 x 32 vector gradients, half of the waves each
    const int o = tid >> 1, type = o / kH, u = o % kH;
    const int q = 4 * (u >> 4) + (u & 3), gg = (u >> 2) & 3;
    float v = 0.0f;
    for (int k = 2 * (tid & 1); k < 2 * (tid & 1) + 2; ++k) {
      const float* r0 = buf + (k * 4 * kQ + type * kQ + q) * kRow + gg * kTrainCols;
#pragma unroll
      for (int j = 0; j < kTrainCols; ++j) v += r0[j];
    }
    v += __shfl_xor(v, 1, kWave);
    const int off = type == 0 ? OFF_W1 : type == 1 ? OFF_B1 : type == 2 ? OFF_B2 : OFF_W3;
    if ((tid & 1) == 0) gp[off + u] = v;
  }
  if (tid == 0) {
    double l = 0.0;
    float v = 0.0f;
    for (int k = 0; k < kTrainWaves; ++k) {
      l += red[k];
      v += red3[k];
    }
    gp[OFF_B3] = v;
    lpart[blockIdx.x] = l;
  }
}

// Sum the block partials (at most kTrainBlocks) in block order, one parameter
// per thread; optionally apply one Adam step (beta1 0.9, beta2 0.999, eps 1e-8)
// and refresh the BF16 copy.  Bound by the latency of the partials' loads, so
// thirty-two are in flight and the parameters are spread over five blocks (17.9 us
// as one block that loaded them one after the other, 4.2 us so).
constexpr int kReduceThreads = 256;
constexpr int kReduceBlocks = (kNParam + kWave + kReduceThreads - 1) / kReduceThreads;

__global__ __launch_bounds__(kReduceThreads) void k_mlp_reduce_adam(
    const float* __restrict__ gpart, const double* __restrict__ lpart, int nblocks, int64_t batch,
    float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
    uint16_t* __restrict__ wb, float lr, float bc1, float bc2, int update,
    float* __restrict__ gsum, float* __restrict__ loss_out) {
  const int p = blockIdx.x * kReduceThreads + threadIdx.x;
  if (p < kNParam) {
    float m0 = 0.0f, v0 = 0.0f, w0 = 0.0f;
    if (update) {
      m0 = m[p];
      v0 = v[p];
      w0 = w[p];
    }
    double sum = 0.0;  // the blocks' parts are added in 64 bits and rounded once
    constexpr int kAhead = 32;
    for (int b0 = 0; b0 < nblocks; b0 += kAhead) {
      float x[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k)  // the row clamped, so that no load waits on a branch
        x[k] = gpart[(int64_t)min(b0 + k, nblocks - 1) * kNParam + p];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) sum += b0 + k < nblocks ? (double)x[k] : 0.0;
    }
    const float g = (float)sum;
    if (gsum) gsum[p] = g;
    if (update) {
      const float mm = 0.9f * m0 + 0.1f * g;
      const float vv = 0.999f * v0 + 0.001f * g * g;
      m[p] = mm;
      v[p] = vv;
      const float wn = w0 - lr * (mm / bc1) / (sqrtf(vv / bc2) + 1e-8f);
      w[p] = wn;
      wb[p] = f32_to_bf16_bits(wn);
    }
  }
  // the loss, by the last block's last wave, which has no parameters
  if (loss_out && blockIdx.x == gridDim.x - 1 && threadIdx.x >= kReduceThreads - kWave) {
    const int lane = threadIdx.x % kWave;
    const double s = wave_sum(lane < nblocks ? lpart[lane] : 0.0);
    if (lane == 0) *loss_out = (float)(s / (double)batch);
  }
}
static_assert(kTrainBlocks <= kWave, "one loss partial per lane");
static_assert(kReduceBlocks * kReduceThreads - kNParam >= kWave, "a wave without parameters");

__global__ void k_to_bf16(const float* __restrict__ w, uint16_t* __restrict__ wb, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) wb[i] = f32_to_bf16_bits(w[i]);
}

// ---- host helpers -------------------------------------------------------------------
inline double eos_energy_host(const Phys& P, double th) {
  if (P.eos == 0) return P.cv * th;
  const double x = P.eos_omega / th;
  return P.eos_n * P.eos_omega * std::exp(-x) / (-std::expm1(-x)) + P.eos_c0 * th;
}

template <typename T>
inline int mlp_alloc(MlpState& s, T** p, size_t count) {
  void* ptr = nullptr;
  if (hipMalloc(&ptr, (count ? count : 1) * sizeof(T)) != hipSuccess) return DPDE_ENOMEM;
  s.allocs.push_back(ptr);
  *p = (T*)ptr;
  return DPDE_OK;
}

inline void mlp_release(MlpState& s) {
  for (void* p : s.allocs) (void)hipFree(p);
  s.allocs.clear();
  s = MlpState{};
}

inline int mlp_ensure_weights(MlpState& s) {
  if (s.w) return DPDE_OK;
  int rc;
  if ((rc = mlp_alloc(s, &s.w, kNParam)) || (rc = mlp_alloc(s, &s.wb, kNParam)) ||
      (rc = mlp_alloc(s, &s.adam_m, kNParam)) || (rc = mlp_alloc(s, &s.adam_v, kNParam)) ||
      (rc = mlp_alloc(s, &s.gsum, kNParam)))
    return rc;
  return DPDE_OK;
}

inline MlpDev mlp_dev(const MlpState& s) {
  return MlpDev{s.w, s.wb, s.norm[0], s.norm[1], s.norm[2], s.norm[3], s.eps_lo, s.eps_hi};
}

// Copy the normalisation into the physics block used by the step kernels.
inline void mlp_attach(MlpState& s, Phys& P) {
  P.mlp_in_c = s.norm[0];
  P.mlp_in_s = s.norm[1];
  P.mlp_out_c = s.norm[2];
  P.mlp_out_s = s.norm[3];
  P.mlp_eps_lo = s.eps_lo;
  P.mlp_eps_hi = s.eps_hi;
}

// 1/theta of the state's internal energies with the handle's theta mode,
// written with a stride (in doubles) into the particle records.
inline void enqueue_theta_mlp(MlpState& s, hipStream_t st, const double* eps, double* invT,
                              int64_t stride, int64_t n, const Phys& P, uint32_t* status) {
  const int mode = s.trained ? P.theta_mode : 0;
  hipLaunchKernelGGL(k_theta<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, eps, invT,
                     stride, (int32_t*)nullptr, n, P, mlp_dev(s), mode, status);
}

inline void launch_theta(MlpState& s, hipStream_t st, const double* eps, double* theta,
                         int32_t* iters, int64_t n, const Phys& P, int mode) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_theta<0>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, eps, theta,
                     (int64_t)1, iters, n, P, mlp_dev(s), mode, (uint32_t*)nullptr);
}

inline int mlp_set(MlpState& s, const Phys& P, const float* w, const double* norm4,
                   std::string& err) {
  (void)P;
  if (mlp_ensure_weights(s)) { err = "allocation failed"; return DPDE_ENOMEM; }
  if (hipMemcpy(s.w, w, kNParam * sizeof(float), hipMemcpyHostToDevice) != hipSuccess) {
    err = "copy failed";
    return DPDE_EHIP;
  }
  hipLaunchKernelGGL(k_to_bf16, dim3((kNParam + 255) / 256), dim3(256), 0, nullptr, s.w, s.wb,
                     kNParam);
  if (hipDeviceSynchronize() != hipSuccess) { err = "conversion failed"; return DPDE_EHIP; }
  for (int k = 0; k < 4; ++k) s.norm[k] = norm4[k];
  // training range of eps implied by the normalisation: x in [-1, 1]
  s.eps_lo = std::exp(norm4[0] - norm4[1]);
  s.eps_hi = std::exp(norm4[0] + norm4[1]);
  s.trained = true;
  return DPDE_OK;
}

inline int mlp_get(MlpState& s, float* w, double* norm4, std::string& err) {
  if (!s.w) { err = "the surrogate has no weights"; return DPDE_EINVAL; }
  if (w && hipMemcpy(w, s.w, kNParam * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess) {
    err = "copy failed";
    return DPDE_EHIP;
  }
  if (norm4)
    for (int k = 0; k < 4; ++k) norm4[k] = s.norm[k];
  return DPDE_OK;
}

inline int mlp_ensure_train_buffers(MlpState& s, int gblocks, int64_t loss_cap) {
  int rc;
  if (s.gblocks < gblocks) {
    if ((rc = mlp_alloc(s, &s.gpart, (size_t)gblocks * kNParam)) ||
        (rc = mlp_alloc(s, &s.lpart, gblocks)))
      return rc;
    s.gblocks = gblocks;
  }
  if (s.loss_cap < loss_cap) {
    if ((rc = mlp_alloc(s, &s.loss, loss_cap))) return rc;
    s.loss_cap = loss_cap;
  }
  return DPDE_OK;
}

inline int mlp_grad(MlpState& s, hipStream_t st, const float* x, const float* t, int64_t n,
                    float* loss, float* grad, std::string& err) {
  if (!s.w) { err = "the surrogate has no weights"; return DPDE_EINVAL; }
  if (n <= 0) { err = "n must be > 0"; return DPDE_EINVAL; }
  const int gb = train_blocks(n);
  if (mlp_ensure_train_buffers(s, gb, 1)) { err = "allocation failed"; return DPDE_ENOMEM; }
  hipLaunchKernelGGL(k_mlp_fwd_bwd, dim3(gb), dim3(kTrainThreads), 0, st, (const float*)s.w, x, t,
                     n, (int64_t)0, n, 1.0f / (float)n, s.gpart, s.lpart);
  hipLaunchKernelGGL(k_mlp_reduce_adam, dim3(kReduceBlocks), dim3(kReduceThreads), 0, st, (const float*)s.gpart,
                     (const double*)s.lpart, gb, n, s.w, s.adam_m, s.adam_v, s.wb, 0.0f, 1.0f,
                     1.0f, 0, s.gsum, s.loss);
  if (hipMemcpyAsync(grad, s.gsum, kNParam * sizeof(float), hipMemcpyDeviceToHost, st) !=
          hipSuccess ||
      hipMemcpyAsync(loss, s.loss, sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess) {
    err = "gradient kernels failed";
    return DPDE_EHIP;
  }
  return DPDE_OK;
}

inline int mlp_eval(MlpState& s, hipStream_t st, const float* x, float* y, int64_t n,
                    std::string& err) {
  if (!s.wb) { err = "the surrogate has no weights"; return DPDE_EINVAL; }
  if (n <= 0) return DPDE_OK;
  hipLaunchKernelGGL(k_mlp_eval, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     (const float*)s.w, (const uint16_t*)s.wb, x, y, n);
  if (hipStreamSynchronize(st) != hipSuccess) { err = "inference kernel failed"; return DPDE_EHIP; }
  return DPDE_OK;
}

template <typename Cfg>
inline int mlp_train(MlpState& s, hipStream_t st, const Phys& P, const Cfg& cfg,
                     float* loss_curve, std::string& err) {
  if (!(cfg.theta_lo > 0 && cfg.theta_hi > cfg.theta_lo) || cfg.nsamples < 1 || cfg.iters < 0 ||
      cfg.batch < 1 || !(cfg.lr > 0)) {
    err = "bad training configuration";
    return DPDE_EINVAL;
  }
  if (mlp_ensure_weights(s)) { err = "allocation failed"; return DPDE_ENOMEM; }
  if (s.nsamp < cfg.nsamples) {
    if (mlp_alloc(s, &s.xs, cfg.nsamples) || mlp_alloc(s, &s.ts, cfg.nsamples)) {
      err = "allocation failed";
      return DPDE_ENOMEM;
    }
    s.nsamp = cfg.nsamples;
  }
  const double elo = eos_energy_host(P, cfg.theta_lo), ehi = eos_energy_host(P, cfg.theta_hi);
  s.norm[0] = 0.5 * (std::log(elo) + std::log(ehi));
  s.norm[1] = 0.5 * (std::log(ehi) - std::log(elo));
  s.norm[2] = 0.5 * (std::log(cfg.theta_lo) + std::log(cfg.theta_hi));
  s.norm[3] = 0.5 * (std::log(cfg.theta_hi) - std::log(cfg.theta_lo));
  s.eps_lo = elo;
  s.eps_hi = ehi;
  hipLaunchKernelGGL(k_mlp_samples, dim3((unsigned)((cfg.nsamples + 255) / 256)), dim3(256), 0, st,
                     (uint64_t)cfg.seed, (int64_t)cfg.nsamples, std::log(cfg.theta_lo),
                     std::log(cfg.theta_hi), P, s.norm[0], s.norm[1], s.norm[2], s.norm[3], s.xs,
                     s.ts);
  // initial weights: N(0, 1.5^2) input layer, N(0, 1) biases, N(0, 1/32) hidden
  std::vector<float> w0(kNParam);
  std::mt19937_64 gen(cfg.seed ^ 0x9E3779B97F4A7C15ull);
  std::normal_distribution<double> nd(0.0, 1.0);
  for (int k = 0; k < kNParam; ++k) {
    double sd;
    if (k < OFF_B1) sd = 1.5;
    else if (k < OFF_W2) sd = 1.0;
    else if (k < OFF_B2) sd = 1.0 / std::sqrt((double)kH);
    else if (k < OFF_W3) sd = 0.0;
    else if (k < OFF_B3) sd = 1.0 / std::sqrt((double)kH);
    else sd = 0.0;
    w0[k] = (float)(sd * nd(gen));
  }
  if (hipMemcpyAsync(s.w, w0.data(), kNParam * sizeof(float), hipMemcpyHostToDevice, st) !=
      hipSuccess) {
    err = "copy failed";
    return DPDE_EHIP;
  }
  (void)hipMemsetAsync(s.adam_m, 0, kNParam * sizeof(float), st);
  (void)hipMemsetAsync(s.adam_v, 0, kNParam * sizeof(float), st);
  hipLaunchKernelGGL(k_to_bf16, dim3((kNParam + 255) / 256), dim3(256), 0, st, (const float*)s.w,
                     s.wb, kNParam);
  const int gb = train_blocks(cfg.batch);
  if (mlp_ensure_train_buffers(s, gb, std::max<int64_t>(1, cfg.iters))) {
    err = "allocation failed";
    return DPDE_ENOMEM;
  }
  double b1p = 1.0, b2p = 1.0;
  for (int64_t it = 0; it < cfg.iters; ++it) {
    b1p *= 0.9;
    b2p *= 0.999;
    // cosine decay of the step size down to 1% of cfg.lr
    const double frac = cfg.iters > 1 ? (double)it / (double)(cfg.iters - 1) : 0.0;
    const double lr = cfg.lr * (0.01 + 0.99 * 0.5 * (1.0 + std::cos(M_PI * frac)));
    const int64_t begin = (it * (int64_t)cfg.batch) % cfg.nsamples;
    hipLaunchKernelGGL(k_mlp_fwd_bwd, dim3(gb), dim3(kTrainThreads), 0, st, (const float*)s.w,
                       (const float*)s.xs, (const float*)s.ts, (int64_t)cfg.nsamples, begin,
                       (int64_t)cfg.batch, 1.0f / (float)cfg.batch, s.gpart, s.lpart);
    hipLaunchKernelGGL(k_mlp_reduce_adam, dim3(kReduceBlocks), dim3(kReduceThreads), 0, st, (const float*)s.gpart,
                       (const double*)s.lpart, gb, (int64_t)cfg.batch, s.w, s.adam_m, s.adam_v,
                       s.wb, (float)lr, (float)(1.0 - b1p), (float)(1.0 - b2p), 1,
                       (float*)nullptr, s.loss + it);
  }
  if (loss_curve && cfg.iters > 0 &&
      hipMemcpyAsync(loss_curve, s.loss, cfg.iters * sizeof(float), hipMemcpyDeviceToHost, st) !=
          hipSuccess) {
    err = "copy failed";
    return DPDE_EHIP;
  }
  if (hipStreamSynchronize(st) != hipSuccess || hipGetLastError() != hipSuccess) {
    err = "training kernels failed";
    return DPDE_EHIP;
  }
  s.trained = true;
  return DPDE_OK;
}

}  // namespace dpde
