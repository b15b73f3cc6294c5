// Training and batch inference of the learned acceptance criterion's network
// (12 -> 64 -> 64 -> 1, ReLU; the same network the walk evaluates).
//
// Forward: the wave-level MFMA routine of mlp_device.h over 64 samples per
// wave.  Loss and gradient (pinball loss at quantile tau on the log10 error
// target): forward, backward and weight gradients of 64 samples per block in one
// kernel on the matrix cores, with the BF16 rounding points of the forward pass
// (weight gradients multiply the rounded activation gradients by the rounded
// activations / inputs; bias gradients use the unrounded activation gradients);
// the blocks' partial sums are added with compensation.
// Adam (Kingma & Ba, bias-corrected) on FP32 master weights, after which the
// BF16 inference image is repacked.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "mlp_device.h"
#include "octgrav_internal.h"

namespace octgrav {
namespace {

using namespace dev;

__global__ void mlp_pack_kernel(const float* __restrict__ P, uint8_t* __restrict__ pk) {
  uint16_t* w1 = reinterpret_cast<uint16_t*>(pk + kPkW1);
  uint16_t* w2 = reinterpret_cast<uint16_t*>(pk + kPkW2);
  float* b1 = reinterpret_cast<float*>(pk + kPkB1);
  float* b2 = reinterpret_cast<float*>(pk + kPkB2);
  uint16_t* w3 = reinterpret_cast<uint16_t*>(pk + kPkW3);
  for (int i = threadIdx.x; i < kMlpH * kMlpInPad; i += blockDim.x) {
    const int j = i / kMlpInPad, k = i % kMlpInPad;
    w1[i] = k < kMlpIn ? (uint16_t)bf16_bits(P[kOffW1 + j * kMlpIn + k]) : (uint16_t)0;
  }
  for (int i = threadIdx.x; i < kMlpH * kMlpH; i += blockDim.x) w2[i] = (uint16_t)bf16_bits(P[kOffW2 + i]);
  for (int i = threadIdx.x; i < kMlpH; i += blockDim.x) {
    b1[i] = P[kOffB1 + i];
    b2[i] = P[kOffB2 + i];
    w3[i] = (uint16_t)bf16_bits(P[kOffW3 + i]);
  }
  if (threadIdx.x == 0) *reinterpret_cast<float*>(pk + kPkB3) = P[kOffB3];
}

// 64 samples per single-wave block.
__global__ __launch_bounds__(64) void mlp_forward_kernel(const uint8_t* __restrict__ pk,
                                                         const float* __restrict__ x, int64_t B,
                                                         float* __restrict__ y) {
  __shared__ uint16_t xs[64 * kMlpInPad];
  const int lane = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * 64, smp = base + lane;
  float f[kMlpIn];
#pragma unroll
  for (int k = 0; k < kMlpIn; ++k) f[k] = smp < B ? x[smp * kMlpIn + k] : 0.f;
  mlp_stage(xs, kMlpInPad, lane, f);
  __syncthreads();
  v4f32 a1[4], a2[4];
  const int quad = lane >> 4;
  const MlpView V = mlp_global(pk);
#pragma unroll 1
  for (int t = 0; t < 4; ++t) {
    const float s = mlp_tile(V, xs, kMlpInPad, t, lane, a1, a2);
    if (quad == t && smp < B) y[smp] = s;
  }
}

// Loss and gradient sums of the samples a block takes, 64 at a time, in one
// kernel; nothing between the inputs and the block's partial sums leaves the
// CU.  Wave w runs the network on samples 16 w ... 16 w + 15 of a chunk
// (mlp_tile), then the backward pass in the same register layout (lane l: sample
// l % 16, units 16 mb + 4 (l / 16) + r): dh2 = (a2 > 0) dL/dy w3, its BF16 rounding
// d2r as the next product's B operand in mlp_tile's contraction order, dh1 = (a1 >
// 0) W2^T d2r as 8 MFMAs against a transposed LDS copy of W2.  The BF16 roundings of
// dh1, d2r, relu(a1) and x go to LDS unit-major, where they are the operands of the
// weight gradients (contraction over the chunk's samples, exact BF16 x BF16
// products, FP32 sums): wave w holds rows 16 w ... 16 w + 15 of dW2 and dW1.  Bias,
// w3 and loss sums stay in registers until the end.
//
// Bound: latency, a few dependent phases per chunk; a mini-batch of 4096 is 64
// blocks of one chunk.  As forward, backward and gradient kernels with the
// activations in global memory (about 1.7 KB per sample each way, and the bias
// sums one sample at a time) the three took 39 us at 4096.
constexpr int kTrLd = 72;  // unit-major row stride (64 samples + 8: 16-byte rows, banks spread)
struct TrainLds {
  // (the operand arrays are read 8 and 16 bytes at a time)
  alignas(16) uint16_t d2[kMlpH * kTrLd], h1[kMlpH * kTrLd], d1[kMlpH * kTrLd], xr[kMlpInPad * kTrLd];
  alignas(16) uint16_t w2t[kMlpH * kW2Ld];  // W2^T, rows padded like the network's copy
  alignas(16) uint16_t xs[64 * kXsLd];
  alignas(16) MlpLds net;
  float w3f[kMlpH];
  float sums[4][3 * kMlpH + 2];
};

__device__ __forceinline__ float row_sum16(float v) {  // over the 16 lanes of a DPP row
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x118, 0xf, 0xf, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x114, 0xf, 0xf, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x112, 0xf, 0xf, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x111, 0xf, 0xf, false));
  return v;  // in lane 15 of the row
}

__global__ __launch_bounds__(256) void mlp_train_kernel(const uint8_t* __restrict__ pk,
                                                        const float* __restrict__ x,
                                                        const float* __restrict__ tgt, int64_t B,
                                                        float tau, float* __restrict__ part) {
  __shared__ __align__(16) TrainLds L;
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 15, quad = lane >> 4;
  const int wave = uni(tid >> 6);
  mlp_load_lds(L.net, pk, tid, 256);
  const uint16_t* w2 = reinterpret_cast<const uint16_t*>(pk + kPkW2);
  for (int i = tid; i < kMlpH * kMlpH; i += 256)  // W2[k][j]: unit k of layer 2, input j
    L.w2t[(i % kMlpH) * kW2Ld + i / kMlpH] = w2[i];
  if (tid < kMlpH)
    L.w3f[tid] = __uint_as_float((uint32_t) reinterpret_cast<const uint16_t*>(pk + kPkW3)[tid] << 16);
  for (int i = tid; i < 64 * 4; i += 256) L.xs[(i / 4) * kXsLd + kMlpIn + i % 4] = 0;
  for (int i = tid; i < (kMlpInPad - kMlpIn) * kTrLd; i += 256) L.xr[kMlpIn * kTrLd + i] = 0;

  v4f32 g2[4], g1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int jb = 0; jb < 4; ++jb) g2[jb] = v4f32{0.f, 0.f, 0.f, 0.f};
  float sb1[16], sb2[16], sw3[16], sb3 = 0.f, sl = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) sb1[i] = sb2[i] = sw3[i] = 0.f;

  for (int64_t base = (int64_t)blockIdx.x * 64; base < B; base += (int64_t)gridDim.x * 64) {
    // inputs, rounded once (by the conversion of the forward pass, which keeps
    // every NaN one); samples past the batch are zero
    for (int i = tid; i < 64 * kMlpIn; i += 256) {
      const int sm = i / kMlpIn, k = i % kMlpIn;
      const uint16_t v = base + sm < B ? (uint16_t)pk_bf16(x[base * kMlpIn + i], 0.f) : (uint16_t)0;
      L.xs[sm * kXsLd + k] = v;
      L.xr[k * kTrLd + sm] = v;
    }
    __syncthreads();
    const MlpView V = mlp_lds(L.net);
    v4f32 a1[4], a2[4];
    const float y = mlp_tile(V, L.xs, kXsLd, wave, lane, a1, a2);
    const int sm = 16 * wave + row;
    const int64_t b = base + sm;
    float dy = 0.f;
    if (b < B) {
      const float r = tgt[b] - y;
      dy = (r > 0.f ? -tau : 1.f - tau) / (float)B;
      if (quad == 0) {
        sl += r > 0.f ? tau * r : (tau - 1.f) * r;
        sb3 += dy;
      }
    }
    uint2 p2[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      const int k0 = 16 * mb + 4 * quad;
      float d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r] = a2[mb][r] > 0.f ? dy * L.w3f[k0 + r] : 0.f;
        sb2[4 * mb + r] += d[r];
        sw3[4 * mb + r] += dy * bf16_round(fmaxf(a2[mb][r], 0.f));
      }
      p2[mb] = make_uint2(pk_bf16(d[0], d[1]), pk_bf16(d[2], d[3]));
      // (a NaN activation counts as inactive here, as in dh1 and dh2)
      const uint2 h = make_uint2(pk_bf16(fmaxf(a1[mb][0], 0.f), fmaxf(a1[mb][1], 0.f)),
                                 pk_bf16(fmaxf(a1[mb][2], 0.f), fmaxf(a1[mb][3], 0.f)));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        L.d2[(k0 + r) * kTrLd + sm] = (uint16_t)((r & 2 ? p2[mb].y : p2[mb].x) >> (16 * (r & 1)));
        L.h1[(k0 + r) * kTrLd + sm] = (uint16_t)((r & 2 ? h.y : h.x) >> (16 * (r & 1)));
      }
    }
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      v4f32 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint16_t* wr = L.w2t + (16 * mb + row) * kW2Ld + 32 * q + 4 * quad;
        const uint2 lo = *reinterpret_cast<const uint2*>(wr);
        const uint2 hi = *reinterpret_cast<const uint2*>(wr + 16);
        const v4u32 av = {lo.x, lo.y, hi.x, hi.y};
        const v4u32 bv = {p2[2 * q].x, p2[2 * q].y, p2[2 * q + 1].x, p2[2 * q + 1].y};
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf16, av),
                                                    __builtin_bit_cast(v8bf16, bv), c, 0, 0, 0);
      }
      const int j0 = 16 * mb + 4 * quad;
      float d[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d[r] = a1[mb][r] > 0.f ? c[r] : 0.f;
        sb1[4 * mb + r] += d[r];
      }
      const uint2 p = make_uint2(pk_bf16(d[0], d[1]), pk_bf16(d[2], d[3]));
#pragma unroll
      for (int r = 0; r < 4; ++r)
        L.d1[(j0 + r) * kTrLd + sm] = (uint16_t)((r & 2 ? p.y : p.x) >> (16 * (r & 1)));
    }
    __syncthreads();
    // Weight gradients over the chunk's samples, two K steps of 32.
    auto op = [&](const uint16_t* m, int blk, int q) {
      return __builtin_bit_cast(v8bf16, *reinterpret_cast<const v4u32*>(m + (16 * blk + row) * kTrLd +
                                                                        32 * q + 8 * quad));
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const v8bf16 a = op(L.d2, wave, q);
#pragma unroll
      for (int jb = 0; jb < 4; ++jb)
        g2[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, op(L.h1, jb, q), g2[jb], 0, 0, 0);
      g1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op(L.d1, wave, q), op(L.xr, 0, q), g1, 0, 0, 0);
    }
    __syncthreads();
  }

  // D layout: rows 16 wave + 4 quad + r, column `row` of each 16-column block
  float* out = part + (int64_t)blockIdx.x * (kMlpParams + 1);
#pragma unroll
  for (int jb = 0; jb < 4; ++jb)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      out[kOffW2 + (16 * wave + 4 * quad + r) * kMlpH + 16 * jb + row] = g2[jb][r];
  if (row < kMlpIn)
#pragma unroll
    for (int r = 0; r < 4; ++r) out[kOffW1 + (16 * wave + 4 * quad + r) * kMlpIn + row] = g1[r];
  // the other sums over a wave's samples, then over the waves in order
  sb3 = row_sum16(sb3);
  sl = row_sum16(sl);
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float v1 = row_sum16(sb1[i]), v2 = row_sum16(sb2[i]), v3 = row_sum16(sw3[i]);
    const int u = 16 * (i >> 2) + 4 * quad + (i & 3);
    if (row == 15) {
      L.sums[wave][u] = v1;
      L.sums[wave][kMlpH + u] = v2;
      L.sums[wave][2 * kMlpH + u] = v3;
    }
  }
  if (lane == 15) {  // quad 0 holds them
    L.sums[wave][3 * kMlpH] = sb3;
    L.sums[wave][3 * kMlpH + 1] = sl;
  }
  __syncthreads();
  if (tid < 3 * kMlpH + 2) {
    const float v = ((L.sums[0][tid] + L.sums[1][tid]) + L.sums[2][tid]) + L.sums[3][tid];
    const int o = tid < kMlpH ? kOffB1 + tid
                  : tid < 2 * kMlpH ? kOffB2 + tid - kMlpH
                  : tid < 3 * kMlpH ? kOffW3 + tid - 2 * kMlpH
                  : tid == 3 * kMlpH ? kOffB3 : kMlpParams;
    out[o] = v;
  }
}

// Sum of the blocks' partial sums, the gradient (also to hgrad, page-locked
// host memory, unless NULL) and the mean loss (FP64, to loss and, unless NULL,
// hloss).  64 parameters per block, four lanes each: every fourth partial
// compensated, the four added in order.
__global__ __launch_bounds__(256) void mlp_grad_reduce_kernel(const float* __restrict__ part,
                                                              int np, int64_t B,
                                                              float* __restrict__ grad,
                                                              double* __restrict__ loss, float* hgrad,
                                                              double* hloss) {
  __shared__ double sh[4][64];
  const int c = threadIdx.x & 63, l = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + c;
  const float* q = part + p;
  if (p == kMlpParams) {  // this lane's column is the loss
    double s = 0.0;
    for (int k = l; k < np; k += 4) s += (double)q[(int64_t)k * (kMlpParams + 1)];
    sh[l][c] = s;
  } else if (p < kMlpParams) {
    float s = 0.f, e = 0.f;
#pragma unroll 4
    for (int k = l; k < np; k += 4) neu_add(s, e, q[(int64_t)k * (kMlpParams + 1)]);
    sh[l][c] = (double)s + (double)e;
  }
  __syncthreads();
  if (l != 0 || p > kMlpParams) return;
  const double s = ((sh[0][c] + sh[1][c]) + sh[2][c]) + sh[3][c];
  if (p == kMlpParams) {
    *loss = s / (double)B;
    if (hloss) *hloss = s / (double)B;
  } else {
    grad[p] = (float)s;
    if (hgrad) hgrad[p] = (float)s;
  }
}

// Adam on the FP32 parameters, and the updated parameter's place in the packed
// BF16 image (whose zero columns the first packing wrote).
__global__ void mlp_adam_kernel(float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                                const float* __restrict__ g, uint8_t* __restrict__ pk, float lr,
                                float b1, float b2, float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= kMlpParams) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float w = P[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  P[i] = w;
  if (i < kOffB1)
    reinterpret_cast<uint16_t*>(pk + kPkW1)[i / kMlpIn * kMlpInPad + i % kMlpIn] = (uint16_t)bf16_bits(w);
  else if (i < kOffW2)
    reinterpret_cast<float*>(pk + kPkB1)[i - kOffB1] = w;
  else if (i < kOffB2)
    reinterpret_cast<uint16_t*>(pk + kPkW2)[i - kOffW2] = (uint16_t)bf16_bits(w);
  else if (i < kOffW3)
    reinterpret_cast<float*>(pk + kPkB2)[i - kOffB2] = w;
  else if (i < kOffB3)
    reinterpret_cast<uint16_t*>(pk + kPkW3)[i - kOffW3] = (uint16_t)bf16_bits(w);
  else
    *reinterpret_cast<float*>(pk + kPkB3) = w;
}

}  // namespace

int launch_mlp_pack(const float* P, void* pk, void* stream) {
  mlp_pack_kernel<<<1, 256, 0, (hipStream_t)stream>>>(P, (uint8_t*)pk);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_mlp_forward(const void* pk, const float* x, int64_t B, float* y, void* stream) {
  if (B <= 0) return 0;
  mlp_forward_kernel<<<(B + 63) / 64, 64, 0, (hipStream_t)stream>>>((const uint8_t*)pk, x, B, y);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Blocks of the training kernel: one per 64 samples up to two per CU; more
// samples are taken in turns.  (The partial sums, 20 KB per block, are read once
// by the reduction.)
static int train_blocks(int64_t B) { return (int)std::min<int64_t>(512, (B + 63) / 64); }

int64_t mlp_train_scratch_floats(int64_t B) { return (int64_t)train_blocks(B) * (kMlpParams + 1); }

int launch_mlp_loss_grad(const void* pk, const float* x, const float* tgt, int64_t B, float tau,
                         float* scratch, float* grad, double* loss, float* hgrad, double* hloss,
                         void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const int nb = train_blocks(B);
  mlp_train_kernel<<<nb, 256, 0, s>>>((const uint8_t*)pk, x, tgt, B, tau, scratch);
  mlp_grad_reduce_kernel<<<(kMlpParams + 1 + 63) / 64, 256, 0, s>>>(scratch, nb, B, grad, loss, hgrad,
                                                                     hloss);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_mlp_adam(float* P, float* m, float* v, const float* g, void* pk, float lr, float b1,
                    float b2, float eps, float c1, float c2, void* stream) {
  mlp_adam_kernel<<<(kMlpParams + 255) / 256, 256, 0, (hipStream_t)stream>>>(
      P, m, v, g, (uint8_t*)pk, lr, b1, b2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace octgrav
