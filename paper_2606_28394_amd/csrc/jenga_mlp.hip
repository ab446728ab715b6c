// Per-contact warm-start network: packing, batch inference and training on gfx950.
//
//  - mlp_pack_kernel: FP32 parameters -> bfloat16 operand layouts (inference blob and the
//    training copies), every weight and bias rounded to bfloat16 once.
//  - mlp_infer_kernel: the network in LDS, one wave per 32 feature rows, the same matrix-core
//    chain the step kernel runs for its contacts.
//  - mlp_grad_kernel: forward and backward of the mean squared error on 64-row chunks, eight
//    waves per workgroup, operands staged in LDS, weight gradients held in matrix-core
//    accumulators across the workgroup's chunks; one partial gradient per workgroup.
//  - mlp_reduce_kernel: partials summed in a fixed order (deterministic), then
//  - mlp_adamw_kernel: decoupled weight decay Adam on the FP32 master parameters.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <string>

#include "../../include/jenga.h"
#include "jenga_device.h"
#include "mlp_device.h"

namespace jg {
namespace mlp {
namespace {

// training copies of the weights (bfloat16 bits), after the inference blob
constexpr int kTrW1t = 0;                       // [128][32]: W1^T with b1 in column 24
constexpr int kTrW2t = kTrW1t + 128 * 32;       // [128][128]: W2^T  (row = output)
constexpr int kTrW2n = kTrW2t + 128 * 128;      // [128][128]: W2    (row = input)
constexpr int kTrW3t = kTrW2n + 128 * 128;      // [16][128]: W3^T, rows 3..15 zero
constexpr int kTrHalfs = kTrW3t + 16 * 128;
constexpr int kTrBias = 132;                    // FP32: b2[128], b3[3], pad (bf16-rounded)
constexpr size_t kPackedBytes = (size_t)kPkUnits * 16 + (size_t)kTrHalfs * 2 + (size_t)kTrBias * 4;

__device__ inline float rbf(float f) { return __uint_as_float(bf16_bits(f) << 16); }

__device__ inline uint16_t w1aug(const float* P, int k, int o) {   // W1 with the bias as input 24
  const float v = k < kFeat ? P[kOffW1 + k * kHidden + o] : (k == kFeat ? P[kOffB1 + o] : 0.f);
  return (uint16_t)bf16_bits(v);
}

__global__ void mlp_pack_kernel(const float* __restrict__ P, uint4* __restrict__ blob) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  uint16_t* pk16 = reinterpret_cast<uint16_t*>(blob);
  float* pkf = reinterpret_cast<float*>(blob);
  // inference blob: one thread per 16-bit slot of the A-operand tiles
  if (tid < (kPkB2 - kPkW1) * 8) {
    const int unit = tid >> 3, j = tid & 7;
    uint16_t v;
    if (unit < kPkW2) {                              // W1 tiles
      const int m = unit >> 6, lane = unit & 63, g = lane >> 4, r = lane & 15;
      v = w1aug(P, 8 * g + j, 16 * m + r);
    } else if (unit < kPkW3) {                       // W2 tiles
      const int u = unit - kPkW2, lane = u & 63, kb = (u >> 6) & 3, mo = u >> 8, g = lane >> 4, r = lane & 15;
      v = (uint16_t)bf16_bits(P[kOffW2 + kappa(kb, g, j) * kHidden + 16 * mo + r]);
    } else {                                         // W3 tiles
      const int u = unit - kPkW3, lane = u & 63, kb = u >> 6, g = lane >> 4, r = lane & 15;
      v = r < kOut ? (uint16_t)bf16_bits(P[kOffW3 + kappa(kb, g, j) * kOut + r]) : (uint16_t)0;
    }
    pk16[tid] = v;
  }
  if (tid < kHidden) pkf[kPkB2 * 4 + tid] = rbf(P[kOffB2 + tid]);        // b2[16mo + 4g + i] in order
  if (tid < 4) pkf[kPkB3 * 4 + tid] = tid < kOut ? rbf(P[kOffB3 + tid]) : 0.f;
  if (tid < kFeat) {
    pkf[kPkMean * 4 + tid] = P[kOffMean + tid];
    pkf[kPkSd * 4 + tid] = P[kOffSd + tid];
  }
  // training copies
  uint16_t* tr = pk16 + kPkUnits * 8;
  if (tid < 128 * 32) { const int o = tid >> 5, k = tid & 31; tr[kTrW1t + tid] = w1aug(P, k, o); }
  if (tid < 128 * 128) {
    const int a = tid >> 7, b = tid & 127;
    tr[kTrW2t + tid] = (uint16_t)bf16_bits(P[kOffW2 + b * kHidden + a]);   // [out a][in b]
    tr[kTrW2n + tid] = (uint16_t)bf16_bits(P[kOffW2 + a * kHidden + b]);   // [in a][out b]
  }
  if (tid < 16 * 128) {
    const int o = tid >> 7, k = tid & 127;
    tr[kTrW3t + tid] = o < kOut ? (uint16_t)bf16_bits(P[kOffW3 + k * kOut + o]) : (uint16_t)0;
  }
  float* trb = reinterpret_cast<float*>(tr + kTrHalfs);
  if (tid < kTrBias) trb[tid] = tid < kHidden ? rbf(P[kOffB2 + tid]) : (tid < kHidden + kOut ? rbf(P[kOffB3 + tid - kHidden]) : 0.f);
}

// Batch inference.  A workgroup keeps the packed network (45 KB) in LDS and its waves walk the rows
// 32 at a time.  The two GELU layers bound it (about 17 VALU instructions per activation, two of them
// at a quarter of the rate): with the weights in LDS a wave needs 114 registers instead of 500, so
// four share a SIMD instead of one (200,003 rows: 35.5 us, from 55).  Chunks are dealt to workgroups
// first and to their waves last, so that a small batch has a SIMD to each wave.
constexpr int kInferWaves = 8;
constexpr int kInferRows = 32;

// a lane's half of a 32-row chunk's row: 16 of the 32 input slots (features, then zeros)
__device__ inline void load_half_row(const float* __restrict__ feats, int row, int n, int half, float f[kRowWords]) {
#pragma unroll
  for (int k = 0; k < kRowWords; ++k)
    f[k] = row < n && kRowWords * half + k < kFeat ? feats[(size_t)row * kFeat + kRowWords * half + k] : 0.f;
}

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ void __launch_bounds__(kInferWaves * 64, 4)
mlp_infer_kernel(const uint4* __restrict__ pk, const float* __restrict__ feats, int n, float* __restrict__ y) {
  __shared__ uint4 net[kPkUnits];
  __shared__ __align__(16) uint32_t rows[kInferWaves][kInferRows * kRowWords];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, half = lane & 1;
  const int nchunks = (n + kInferRows - 1) / kInferRows, stride = gridDim.x * kInferWaves;
  int c = blockIdx.x + gridDim.x * wave;
  float f[kRowWords];
  load_half_row(feats, c < nchunks ? c * kInferRows + (lane >> 1) : n, n, half, f);
  for (int k = threadIdx.x; k < kPkUnits; k += kInferWaves * 64) net[k] = pk[k];
  __syncthreads();
  uint32_t* const xs = rows[wave];
  const float* const mean = reinterpret_cast<const float*>(net + kPkMean);
  const float* const sd = reinterpret_cast<const float*>(net + kPkSd);
  for (; c < nchunks; c += stride) {
#pragma unroll
    for (int k = 0; k < kRowWords; k += 2) {
      const int q = kRowWords * half + k;
      uint32_t w = q == kFeat ? pack2(1.f, 0.f) : 0u;
      if (q < kFeat) w = pack2((f[k] - mean[q]) / sd[q], (f[k + 1] - mean[q + 1]) / sd[q + 1]);
      xs[(lane >> 1) * kRowWords + (q >> 1)] = w;
    }
    wave_fence();
    // the next chunk's features are on their way while this one is worked
    load_half_row(feats, c + stride < nchunks ? (c + stride) * kInferRows + (lane >> 1) : n, n, half, f);
    f32x4 out[kInferRows / 16];
    infer_chunk<kInferRows / 16>(net, xs, lane, out);
    if (lane < 16) {
#pragma unroll
      for (int t = 0; t < kInferRows / 16; ++t) {
        const int r = c * kInferRows + 16 * t + lane;
        if (r < n)
          for (int o = 0; o < kOut; ++o) y[(size_t)r * kOut + o] = out[t][o];
      }
    }
    wave_fence();
  }
}

// ------------------------------------------------------------------------------------------------
// training: forward + backward on 64-row chunks
// ------------------------------------------------------------------------------------------------
// A workgroup's chunk is a chain of seven short phases between barriers, bound by latency (loads, LDS
// and the barriers), not by its matrix products: the shorter each wave's part, the better.  Eight
// waves each own 16 hidden units of either layer; every global load is in flight before the first
// phase needs one, and the next chunk's during this one.  A training step of 8,192 rows (128
// workgroups, one chunk each) takes 21.8 us, from 56.7 with four waves and one thread per column in
// the reduction; 777 rows 17.3 us, from 26.9.
constexpr int kTrainWaves = kHidden / 16;   // wave w owns hidden units 16 w to 16 w + 15 of either layer
constexpr int kTrainThreads = kTrainWaves * 64;
// LDS row strides in 16-bit units (rows padded by 16 bytes against bank conflicts)
constexpr int kS128 = 136, kS64 = 72, kS32 = 40;
struct TrainLds {
  uint16_t X[64 * kS32];      // [p][k]  inputs (bias column 24)
  uint16_t Xt[32 * kS64];     // [k][p]
  uint16_t H1[64 * kS128];    // [p][h]
  uint16_t H1t[128 * kS64];   // [h][p]
  uint16_t H2[64 * kS128];
  uint16_t H2t[128 * kS64];
  uint16_t dZ2[64 * kS128];   // [p][h]
  uint16_t dZ2t[128 * kS64];  // [h][p]
  uint16_t dZ1t[128 * kS64];  // [h][p]
  uint16_t dYt[16 * kS64];    // [o][p], rows 3..15 zero
  float dY[64 * 4];           // [p][o]
  float T[64 * 4];            // targets
  float loss[4];
};

__device__ inline bf16x8 lds8(const uint16_t* base) { return as_bf16x8(*reinterpret_cast<const uint4*>(base)); }
// four rows p = 16 pt + 4 g + i of column h of a result tile, as bfloat16: into the [h][p] copy (one
// 8-byte store), and with put_tile also into the [p][h] copy
__device__ inline void put_column(uint16_t* t, int pt, int h, int g, float v0, float v1, float v2, float v3) {
  *reinterpret_cast<uint2*>(t + h * kS64 + 16 * pt + 4 * g) = make_uint2(pack2(v0, v1), pack2(v2, v3));
}
__device__ inline void put_tile(uint16_t* rows, uint16_t* t, int pt, int h, int g, float v0, float v1, float v2, float v3) {
  const uint32_t lo = pack2(v0, v1), hi = pack2(v2, v3);
  *reinterpret_cast<uint2*>(t + h * kS64 + 16 * pt + 4 * g) = make_uint2(lo, hi);
  uint16_t* q = rows + (16 * pt + 4 * g) * kS128 + h;
  q[0] = (uint16_t)lo;
  q[kS128] = (uint16_t)(lo >> 16);
  q[2 * kS128] = (uint16_t)hi;
  q[3 * kS128] = (uint16_t)(hi >> 16);
}
__device__ inline bf16x8 glb8(const uint16_t* base) { return as_bf16x8(*reinterpret_cast<const uint4*>(base)); }

__global__ void __launch_bounds__(kTrainThreads, 1)
mlp_grad_kernel(const float* __restrict__ P, const uint4* __restrict__ pk, const float* __restrict__ feats,
                const float* __restrict__ targets, int n, float* __restrict__ partial) {
  extern __shared__ __align__(16) unsigned char smem[];
  TrainLds& S = *reinterpret_cast<TrainLds*>(smem);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 4, r = lane & 15;
  const uint16_t* tr = reinterpret_cast<const uint16_t*>(pk) + kPkUnits * 8;
  const float* trb = reinterpret_cast<const float*>(tr + kTrHalfs);
  const float inv_rows = 1.f / (3.f * (float)n);

  // persistent accumulators: dW1aug tiles (k-tile kt, h-tile w), dW2 tiles (i-tile w, h-tile ht),
  // dW3 tile (h-tile w), db2 / db3 per lane
  f32x4 aW1[2], aW2[8], aW3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 2; ++a) aW1[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 8; ++a) aW2[a] = f32x4{0.f, 0.f, 0.f, 0.f};
  float db2 = 0.f, db3 = 0.f, lsum = 0.f;

  // A chunk's inputs and targets: a thread has one input column, and every load is unconditional (rows
  // clamped to the last), so that all are in flight at once.
  constexpr int kStagePasses = kChunk * 32 / kTrainThreads;
  const int sk = tid & 31, sp = tid >> 5;   // the thread's input column, and its row of each staging pass
  const float smean = reinterpret_cast<const float*>(pk + kPkMean)[min(sk, kFeat - 1)];
  const float ssd = reinterpret_cast<const float*>(pk + kPkSd)[min(sk, kFeat - 1)];
  const int tp = min(tid / 3, kChunk - 1), to = tid % 3;
  float x[kStagePasses], tg = 0.f;
  auto fetch = [&](int c) {
    const int64_t row0 = (int64_t)c * kChunk;
#pragma unroll
    for (int e = 0; e < kStagePasses; ++e)
      x[e] = feats[min(row0 + kTrainThreads / 32 * e + sp, (int64_t)n - 1) * kFeat + min(sk, kFeat - 1)];
    tg = targets[min(row0 + tp, (int64_t)n - 1) * kOut + to];
  };
  fetch(blockIdx.x);
  // the wave's weights
  const int h0 = 16 * wave;
  const bf16x8 w1 = glb8(tr + kTrW1t + (h0 + r) * 32 + 8 * g);
  const float bias2 = trb[h0 + r], bias3 = r < kOut ? trb[kHidden + r] : 0.f;
  bf16x8 w2t[4], w2n[4], w3t[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    w2t[kb] = glb8(tr + kTrW2t + (h0 + r) * 128 + 32 * kb + 8 * g);
    w3t[kb] = glb8(tr + kTrW3t + r * 128 + 32 * kb + 8 * g);
    w2n[kb] = glb8(tr + kTrW2n + (h0 + r) * 128 + 32 * kb + 8 * g);
  }
  float w3[3];
#pragma unroll
  for (int o = 0; o < 3; ++o) w3[o] = rbf(P[kOffW3 + (h0 + r) * 3 + o]);

  const int nchunks = (n + kChunk - 1) / kChunk;
  for (int c = blockIdx.x; c < nchunks; c += gridDim.x) {
    // ---- stage inputs and targets (padding rows are zero: no bias input either) ----
#pragma unroll
    for (int e = 0; e < kStagePasses; ++e) {
      const int p = kTrainThreads / 32 * e + sp;
      float v = sk < kFeat ? (x[e] - smean) / ssd : (sk == kFeat ? 1.f : 0.f);
      if (c * kChunk + p >= n) v = 0.f;
      const uint16_t b = (uint16_t)bf16_bits(v);
      S.X[p * kS32 + sk] = b;
      S.Xt[sk * kS64 + p] = b;
    }
    if (tid < 3 * kChunk) S.T[tp * 4 + to] = c * kChunk + tp < n ? tg : 0.f;
    __syncthreads();
    fetch(c + gridDim.x);   // the next chunk's rows are on their way while this one is worked

    // ---- forward layer 1: Z1[p][h] for the wave's h-tile ----
    f32x4 z1[4], z2[4];
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
      const bf16x8 a = lds8(S.X + (16 * pt + r) * kS32 + 8 * g);
      z1[pt] = mfma(a, w1, f32x4{0.f, 0.f, 0.f, 0.f});
      put_tile(S.H1, S.H1t, pt, h0 + r, g, gelu(z1[pt][0]), gelu(z1[pt][1]), gelu(z1[pt][2]), gelu(z1[pt][3]));
    }
    __syncthreads();
    // ---- forward layer 2 ----
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) z2[pt] = f32x4{bias2, bias2, bias2, bias2};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) {
        const bf16x8 a = lds8(S.H1 + (16 * pt + r) * kS128 + 32 * kb + 8 * g);
        z2[pt] = mfma(a, w2t[kb], z2[pt]);
      }
#pragma unroll
    for (int pt = 0; pt < 4; ++pt)
      put_tile(S.H2, S.H2t, pt, h0 + r, g, gelu(z2[pt][0]), gelu(z2[pt][1]), gelu(z2[pt][2]), gelu(z2[pt][3]));
    __syncthreads();
    // ---- output layer and loss: wave w < 4 owns rows 16w..16w+15 ----
    if (wave < 4) {
      f32x4 y = f32x4{bias3, bias3, bias3, bias3};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const bf16x8 a = lds8(S.H2 + (16 * wave + r) * kS128 + 32 * kb + 8 * g);
        y = mfma(a, w3t[kb], y);
      }
      // lane (g, r) holds y[p = 16w + 4g + i][o = r]
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = 16 * wave + 4 * g + i;
        float d = 0.f;
        if (r < kOut && c * kChunk + p < n) {
          const float e = y[i] - S.T[p * 4 + r];
          lsum += e * e;
          d = 2.f * e * inv_rows;
        }
        if (r < kOut) S.dY[p * 4 + r] = d;
        S.dYt[r * kS64 + p] = (uint16_t)bf16_bits(d);
        db3 += d;
      }
    }
    __syncthreads();
    // ---- dZ2 = (dY W3^T) * gelu'(z2), same tiles as layer 2 ----
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
      float dz[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int p = 16 * pt + 4 * g + i;
        const float dh = S.dY[p * 4] * w3[0] + S.dY[p * 4 + 1] * w3[1] + S.dY[p * 4 + 2] * w3[2];
        dz[i] = dh * gelu_grad(z2[pt][i]);
        db2 += dz[i];
      }
      put_tile(S.dZ2, S.dZ2t, pt, h0 + r, g, dz[0], dz[1], dz[2], dz[3]);
    }
    __syncthreads();
    // ---- dW3[h][o] += H2t[h][:] . dYt[o][:] ----
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const bf16x8 a = lds8(S.H2t + (h0 + r) * kS64 + 32 * kb + 8 * g);
      const bf16x8 b = lds8(S.dYt + r * kS64 + 32 * kb + 8 * g);
      aW3 = mfma(a, b, aW3);
    }
    // ---- dZ1 = (dZ2 W2^T) * gelu'(z1), same tiles as layer 1 ----
    {
      f32x4 acc[4];
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) acc[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
          const bf16x8 a = lds8(S.dZ2 + (16 * pt + r) * kS128 + 32 * kb + 8 * g);
          acc[pt] = mfma(a, w2n[kb], acc[pt]);
        }
#pragma unroll
      for (int pt = 0; pt < 4; ++pt)
        put_column(S.dZ1t, pt, h0 + r, g, acc[pt][0] * gelu_grad(z1[pt][0]), acc[pt][1] * gelu_grad(z1[pt][1]),
                   acc[pt][2] * gelu_grad(z1[pt][2]), acc[pt][3] * gelu_grad(z1[pt][3]));
    }
    __syncthreads();
    // ---- dW2[i][h] += H1t[i][:] . dZ2t[h][:];  dW1aug[k][i] += Xt[k][:] . dZ1t[i][:] ----
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const bf16x8 a = lds8(S.H1t + (h0 + r) * kS64 + 32 * kb + 8 * g);
#pragma unroll
      for (int ht = 0; ht < 8; ++ht) {
        const bf16x8 b = lds8(S.dZ2t + (16 * ht + r) * kS64 + 32 * kb + 8 * g);
        aW2[ht] = mfma(a, b, aW2[ht]);
      }
      const bf16x8 b1 = lds8(S.dZ1t + (h0 + r) * kS64 + 32 * kb + 8 * g);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const bf16x8 a1 = lds8(S.Xt + (16 * kt + r) * kS64 + 32 * kb + 8 * g);
        aW1[kt] = mfma(a1, b1, aW1[kt]);
      }
    }
    __syncthreads();
  }

  // ---- write this workgroup's partial gradient ----
  float* out = partial + (size_t)blockIdx.x * (kTrainable + 1);
  // dW1aug tile (kt, h-tile w): lane holds rows k = 16kt + 4g + i, column h = 16w + r
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 16 * kt + 4 * g + i, h = h0 + r;
      if (k < kFeat) out[kOffW1 + k * kHidden + h] = aW1[kt][i];
      else if (k == kFeat) out[kOffB1 + h] = aW1[kt][i];
    }
#pragma unroll
  for (int ht = 0; ht < 8; ++ht)
#pragma unroll
    for (int i = 0; i < 4; ++i) out[kOffW2 + (h0 + 4 * g + i) * kHidden + 16 * ht + r] = aW2[ht][i];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (r < kOut) out[kOffW3 + (h0 + 4 * g + i) * kOut + r] = aW3[i];
  // db2: lanes (g, r) of one wave hold partial sums of the same column; fold the 4 groups
  {
    float s = db2;
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (g == 0) out[kOffB2 + h0 + r] = s;
  }
  if (wave < 4) {
    float s = db3;
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    // every wave saw its own rows: combine the four waves through LDS
    if (g == 0 && r < kOut) S.dY[wave * 4 + r] = s;
    float l = lsum;
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off);
    if (lane == 0) S.loss[wave] = l;
  }
  __syncthreads();
  if (tid < kOut) out[kOffB3 + tid] = S.dY[tid] + S.dY[4 + tid] + S.dY[8 + tid] + S.dY[12 + tid];
  if (tid == 0) out[kTrainable] = S.loss[0] + S.loss[1] + S.loss[2] + S.loss[3];
}

// Sums of the workgroups' partial gradients: a workgroup takes 64 columns, its waves the partials
// k = w, w + kReduceWaves, ..., so that every load of a column is in flight at once (128 partials of
// 80 KB: 4.6 us, from 30.5 with one thread walking each column); the waves' sums are folded in a
// fixed order (deterministic).  Returns in the first wave.
constexpr int kReduceWaves = 16;
__device__ inline float reduce_column(const float* __restrict__ partial, int nparts, int i, float* sh) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float s = 0.f;
  if (i <= kTrainable) {
#pragma unroll 8
    for (int k = wave; k < nparts; k += kReduceWaves) s += partial[(size_t)k * (kTrainable + 1) + i];
  }
  sh[wave * 64 + lane] = s;
  __syncthreads();
  s = 0.f;
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < kReduceWaves; ++w) s += sh[w * 64 + lane];
  }
  return s;
}

__global__ void __launch_bounds__(kReduceWaves * 64)
mlp_reduce_kernel(const float* __restrict__ partial, int nparts, int n, float* __restrict__ grad,
                  float* __restrict__ loss) {
  __shared__ float sh[kReduceWaves * 64];
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const float s = reduce_column(partial, nparts, i, sh);
  if (threadIdx.x >= 64) return;
  if (i < kTrainable) grad[i] = s;
  else if (i == kTrainable && loss) *loss = s / (3.f * (float)n);
}

__device__ inline void adamw_param(int i, float gi, float* __restrict__ P, float* __restrict__ m, float* __restrict__ v,
                                   float lr, float b1, float b2, float eps, float wd, float c1, float c2) {
  float p = P[i] * (1.f - lr * wd);
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  P[i] = p;
}

__global__ void mlp_adamw_kernel(float* __restrict__ P, const float* __restrict__ grad, float* __restrict__ m,
                                 float* __restrict__ v, float lr, float b1, float b2, float eps, float wd,
                                 float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kTrainable) adamw_param(i, grad[i], P, m, v, lr, b1, b2, eps, wd, c1, c2);
}

// Where parameter i goes in the packed copies, and its rounded value there (mlp_pack_kernel's layout,
// by parameter instead of by slot; the slots that no parameter fills are zero since the first pack)
__device__ inline void pack_param(uint4* blob, int i, float p) {
  uint16_t* pk16 = reinterpret_cast<uint16_t*>(blob);
  float* pkf = reinterpret_cast<float*>(blob);
  uint16_t* tr = pk16 + kPkUnits * 8;
  float* trb = reinterpret_cast<float*>(tr + kTrHalfs);
  const uint16_t b = (uint16_t)bf16_bits(p);
  if (i < kOffW2) {                                  // W1 and, as input 24, b1
    const int k = i >> 7, h = i & 127;
    pk16[(kPkW1 + (h >> 4) * 64 + (k >> 3) * 16 + (h & 15)) * 8 + (k & 7)] = b;
    tr[kTrW1t + h * 32 + k] = b;
  } else if (i < kOffB2) {
    const int in = (i - kOffW2) >> 7, out = (i - kOffW2) & 127;
    const int kb = in >> 5, g = (in >> 2) & 3, j = 4 * ((in >> 4) & 1) + (in & 3);   // kappa(kb, g, j) = in
    pk16[(kPkW2 + ((out >> 4) * 4 + kb) * 64 + g * 16 + (out & 15)) * 8 + j] = b;
    tr[kTrW2t + out * 128 + in] = b;
    tr[kTrW2n + in * 128 + out] = b;
  } else if (i < kOffW3) {
    pkf[kPkB2 * 4 + i - kOffB2] = rbf(p);
    trb[i - kOffB2] = rbf(p);
  } else if (i < kOffB3) {
    const int in = (i - kOffW3) / kOut, o = (i - kOffW3) % kOut;
    const int kb = in >> 5, g = (in >> 2) & 3, j = 4 * ((in >> 4) & 1) + (in & 3);
    pk16[(kPkW3 + kb * 64 + g * 16 + o) * 8 + j] = b;
    tr[kTrW3t + o * 128 + in] = b;
  } else if (i < kOffMean) {
    pkf[kPkB3 * 4 + i - kOffB3] = rbf(p);
    trb[kHidden + i - kOffB3] = rbf(p);
  } else if (i < kOffSd) {
    pkf[kPkMean * 4 + i - kOffMean] = p;
  } else {
    pkf[kPkSd * 4 + i - kOffSd] = p;
  }
}

// The rest of a training step in one launch: the gradient's sums, AdamW and the packed copies, each
// parameter by the thread that summed its column (three dependent launches of 3 to 5 us otherwise).
__global__ void __launch_bounds__(kReduceWaves * 64)
mlp_update_kernel(const float* __restrict__ partial, int nparts, int n, float* __restrict__ grad, float* __restrict__ loss,
                  float* __restrict__ P, uint4* __restrict__ blob, float* __restrict__ m, float* __restrict__ v, float lr,
                  float b1, float b2, float eps, float wd, float c1, float c2) {
  __shared__ float sh[kReduceWaves * 64];
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const float s = reduce_column(partial, nparts, i, sh);
  if (threadIdx.x >= 64 || i >= kParams) return;
  if (i == kTrainable && loss) *loss = s / (3.f * (float)n);
  if (i < kTrainable) {
    grad[i] = s;
    adamw_param(i, s, P, m, v, lr, b1, b2, eps, wd, c1, c2);
  }
  pack_param(blob, i, P[i]);
}

int grad_blocks(int n) {
  const int nchunks = (n + kChunk - 1) / kChunk;
  return nchunks < 256 ? (nchunks > 0 ? nchunks : 1) : 256;
}

}  // namespace

size_t packed_bytes() { return kPackedBytes; }

hipError_t launch_pack(const float* params, void* packed, hipStream_t s) {
  constexpr int threads = (kPkB2 - kPkW1) * 8 > 128 * 128 ? (kPkB2 - kPkW1) * 8 : 128 * 128;
  hipLaunchKernelGGL(mlp_pack_kernel, dim3((threads + 255) / 256), dim3(256), 0, s, params, (uint4*)packed);
  return hipGetLastError();
}

hipError_t launch_infer(const void* packed, const float* feats, int n, float* y, hipStream_t s) {
  const int nchunks = (n + kInferRows - 1) / kInferRows;
  if (nchunks == 0) return hipSuccess;
  const int grid = nchunks < 512 ? nchunks : 512;   // two resident workgroups on each CU
  hipLaunchKernelGGL(mlp_infer_kernel, dim3(grid), dim3(kInferWaves * 64), 0, s, (const uint4*)packed, feats, n, y);
  return hipGetLastError();
}

size_t grad_workspace_bytes(int n) { return (size_t)grad_blocks(n) * (kTrainable + 1) * sizeof(float); }

// the partial gradients of `blocks` workgroups into part
hipError_t launch_partials(const float* params, const void* packed, const float* feats, const float* targets, int n,
                           float* part, int blocks, hipStream_t s) {
  // the kernel's dynamic-LDS limit, once per device (the current one)
  constexpr int kMaxDevices = 64;
  static std::mutex attr_mutex;
  static bool attr[kMaxDevices] = {};
  int dev = 0;
  if (hipError_t e = hipGetDevice(&dev)) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  {
    std::lock_guard<std::mutex> lock(attr_mutex);
    if (!attr[dev]) {
      hipError_t e = hipFuncSetAttribute((const void*)mlp_grad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)sizeof(TrainLds));
      if (e != hipSuccess) return e;
      attr[dev] = true;
    }
  }
  hipLaunchKernelGGL(mlp_grad_kernel, dim3(blocks), dim3(kTrainThreads), sizeof(TrainLds), s, params,
                     (const uint4*)packed, feats, targets, n, part);
  return hipGetLastError();
}

hipError_t launch_grad(const float* params, const void* packed, const float* feats, const float* targets, int n,
                       float* grad, float* loss, void* workspace, hipStream_t s) {
  const int blocks = grad_blocks(n);
  float* part = (float*)workspace;
  if (hipError_t e = launch_partials(params, packed, feats, targets, n, part, blocks, s)) return e;
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3((kTrainable + 1 + 63) / 64), dim3(kReduceWaves * 64), 0, s, part, blocks, n,
                     grad, loss);
  return hipGetLastError();
}

hipError_t launch_train_step(float* params, void* packed, const float* feats, const float* targets, int n, float* grad,
                             float* loss, void* workspace, float* m, float* v, int step, float lr, float b1, float b2,
                             float eps, float wd, hipStream_t s) {
  const int blocks = grad_blocks(n);
  float* part = (float*)workspace;
  if (hipError_t e = launch_partials(params, packed, feats, targets, n, part, blocks, s)) return e;
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(mlp_update_kernel, dim3((kParams + 63) / 64), dim3(kReduceWaves * 64), 0, s, part, blocks, n, grad, loss,
                     params, (uint4*)packed, m, v, lr, b1, b2, eps, wd, c1, c2);
  return hipGetLastError();
}

hipError_t launch_adamw(float* params, const float* grad, float* m, float* v, int step, float lr, float b1, float b2,
                        float eps, float wd, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(mlp_adamw_kernel, dim3((kTrainable + 255) / 256), dim3(256), 0, s, params, grad, m, v, lr, b1,
                     b2, eps, wd, c1, c2);
  return hipGetLastError();
}

}  // namespace mlp
}  // namespace jg

// Scratch of jg_mlp_grad_noalloc: the per-workgroup partial gradients of one call, at most
// kGradScratchParts rows of JG_MLP_TRAINABLE + 1 floats (256 x 20100 x 4 B = 20.6 MB; the
// gradient launch never uses more workgroups).  Each device the library runs on holds its own
// copy until the process ends.  Every row a call reads is written earlier in the same call.
constexpr int kGradScratchParts = 256;
static __device__ __align__(256) float scratch[(size_t)kGradScratchParts * (JG_MLP_TRAINABLE + 1)];

// ------------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------------
namespace {
int32_t hip_status(hipError_t e, const char* what) {
  if (e == hipSuccess) return JG_OK;
  return jg::set_error(JG_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// The device address of `scratch` on the current device, looked up on the first call there
// (the array's name is only a host-side stand-in; kernels get this address).
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mutex;
float* g_scratch_ptr[kScratchDevices] = {};

int32_t scratch_on_current_device(float** out) {
  int dev = 0;
  if (hipError_t e = hipGetDevice(&dev)) return hip_status(e, "jg_mlp_grad_noalloc: hipGetDevice");
  if (dev < 0 || dev >= kScratchDevices) return jg::set_error(JG_EDEVICE, "jg_mlp_grad_noalloc: device ordinal out of range");
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)))
      return hip_status(e, "jg_mlp_grad_noalloc: hipGetSymbolAddress(scratch)");
    if (!p) return jg::set_error(JG_EDEVICE, "jg_mlp_grad_noalloc: no device address for the scratch array");
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return JG_OK;
}
}  // namespace

extern "C" {

int32_t jg_mlp_packed_bytes(size_t* bytes) {
  if (!bytes) return jg::set_error(JG_EINVAL, "jg_mlp_packed_bytes: null pointer");
  *bytes = jg::mlp::packed_bytes();
  return JG_OK;
}

int32_t jg_mlp_pack(const float* params, void* packed, void* stream) {
  if (!params || !packed) return jg::set_error(JG_EINVAL, "jg_mlp_pack: null pointer");
  return hip_status(jg::mlp::launch_pack(params, packed, (hipStream_t)stream), "jg_mlp_pack");
}

int32_t jg_mlp_forward(const void* packed, const float* feats, int32_t n, float* y, void* stream) {
  if (n < 0) return jg::set_error(JG_EINVAL, "jg_mlp_forward: negative row count");
  if (n == 0) return JG_OK;
  if (!packed || !feats || !y) return jg::set_error(JG_EINVAL, "jg_mlp_forward: null pointer");
  return hip_status(jg::mlp::launch_infer(packed, feats, n, y, (hipStream_t)stream), "jg_mlp_forward");
}

int32_t jg_mlp_grad_workspace_bytes(int32_t n, size_t* bytes) {
  if (n < 0 || !bytes) return jg::set_error(JG_EINVAL, "jg_mlp_grad_workspace_bytes: bad argument");
  *bytes = jg::mlp::grad_workspace_bytes(n);
  return JG_OK;
}

int32_t jg_mlp_grad(const float* params, const void* packed, const float* feats, const float* targets, int32_t n,
                    float* grad, float* loss, void* workspace, size_t workspace_bytes, void* stream) {
  if (n <= 0) return jg::set_error(JG_EINVAL, "jg_mlp_grad: the batch must hold at least one row");
  if (!params || !packed || !feats || !targets || !grad || !workspace)
    return jg::set_error(JG_EINVAL, "jg_mlp_grad: null pointer");
  if (workspace_bytes < jg::mlp::grad_workspace_bytes(n))
    return jg::set_error(JG_EINVAL, "jg_mlp_grad: workspace smaller than jg_mlp_grad_workspace_bytes(n)");
  return hip_status(jg::mlp::launch_grad(params, packed, feats, targets, n, grad, loss, workspace, (hipStream_t)stream),
                    "jg_mlp_grad");
}

int32_t jg_mlp_grad_noalloc(const float* params, const void* packed, const float* feats, const float* targets,
                            int32_t n, float* grad, float* loss, void* stream) {
  if (n <= 0) return jg::set_error(JG_EINVAL, "jg_mlp_grad_noalloc: the batch must hold at least one row");
  if (!params || !packed || !feats || !targets || !grad)
    return jg::set_error(JG_EINVAL, "jg_mlp_grad_noalloc: null pointer");
  if (jg::mlp::grad_workspace_bytes(n) > sizeof(scratch))
    return jg::set_error(JG_ECAPACITY, "jg_mlp_grad_noalloc: the batch needs " +
                                       std::to_string(jg::mlp::grad_workspace_bytes(n)) +
                                       " bytes of partial sums, more than the static scratch holds (" +
                                       std::to_string(sizeof(scratch)) + ")");
  float* ws = nullptr;
  if (int32_t r = scratch_on_current_device(&ws)) return r;
  return hip_status(jg::mlp::launch_grad(params, packed, feats, targets, n, grad, loss, ws, (hipStream_t)stream),
                    "jg_mlp_grad_noalloc");
}

int32_t jg_mlp_train_step(float* params, void* packed, const float* feats, const float* targets, int32_t n, float* grad,
                          float* loss, void* workspace, size_t workspace_bytes, float* m, float* v, int32_t step,
                          float lr, float beta1, float beta2, float eps, float weight_decay, void* stream) {
  if (n <= 0) return jg::set_error(JG_EINVAL, "jg_mlp_train_step: the batch must hold at least one row");
  if (!params || !packed || !feats || !targets || !grad || !workspace || !m || !v)
    return jg::set_error(JG_EINVAL, "jg_mlp_train_step: null pointer");
  if (workspace_bytes < jg::mlp::grad_workspace_bytes(n))
    return jg::set_error(JG_EINVAL, "jg_mlp_train_step: workspace smaller than jg_mlp_grad_workspace_bytes(n)");
  if (step < 1) return jg::set_error(JG_EINVAL, "jg_mlp_train_step: step counts from 1");
  return hip_status(jg::mlp::launch_train_step(params, packed, feats, targets, n, grad, loss, workspace, m, v, step, lr,
                                               beta1, beta2, eps, weight_decay, (hipStream_t)stream),
                    "jg_mlp_train_step");
}

int32_t jg_mlp_adamw(float* params, const float* grad, float* m, float* v, int32_t step, float lr, float beta1,
                     float beta2, float eps, float weight_decay, void* stream) {
  if (!params || !grad || !m || !v) return jg::set_error(JG_EINVAL, "jg_mlp_adamw: null pointer");
  if (step < 1) return jg::set_error(JG_EINVAL, "jg_mlp_adamw: step counts from 1");
  return hip_status(jg::mlp::launch_adamw(params, grad, m, v, step, lr, beta1, beta2, eps, weight_decay,
                                          (hipStream_t)stream),
                    "jg_mlp_adamw");
}

}  // extern "C"
