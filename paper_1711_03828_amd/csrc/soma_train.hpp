// soma_train.hpp -- training of the learned proposal's network on the matrix
// cores: forward, Gaussian negative log-likelihood of observed displacements,
// back-propagation and Adam, all with BF16 MFMA inputs and FP32 accumulation.
//
// A block of four waves takes chunks of 64 samples, 16 per wave.  Every matrix
// product is a v_mfma_f32_16x16x32_bf16 tile: the forward and the error
// propagation contract over units (a wave's samples stay in its own rows of a
// sample-major LDS tile, so the layers need no block barrier), the weight
// gradients contract over the 64 samples of the chunk (unit-major, transposed
// LDS tiles; wave w owns the 16 input units 16 w .. of every gradient).
// Gradients accumulate in registers over all chunks of the block and are
// written once as a partial; a second kernel sums the partials in a fixed
// order and applies Adam to the FP32 master parameters.
#pragma once

#include "soma_mlp.hpp"

namespace soma {

constexpr int kTStride = 72;  // bf16 per row of a transposed (unit-major) tile

struct TrainArgs {
  const float *params;   // FP32 blob
  const float *feat;     // [n][60] raw features
  const float *target;   // [n][3] displacements
  uint32_t n;
  uint32_t vec4;         // params and feat are 16-byte aligned
  HeadArgs head;
  float *partials;       // [blocks][kPSize] gradient partials (sums over samples)
  float *loss_partials;  // [blocks]
};

__device__ __forceinline__ bf16x8 lds8(const __bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Four consecutive floats, as one 16-byte load where the base is aligned (the
// offsets used are multiples of four).
__device__ __forceinline__ f32x4 load_f4(const float *p, uint32_t vec4) {
  if (vec4) return *reinterpret_cast<const f32x4 *>(p);
  return f32x4{p[0], p[1], p[2], p[3]};
}

// The weights of a block as BF16 tiles: W1 (inputs 60..63 zero), W2, W2
// transposed, W3 (rows >= 6 zero) and W3 transposed ([hidden][8], outputs >= 6
// zero), with the FP32 standardisation and biases.
struct alignas(16) TrainLds {
  __bf16 w1[64 * kTStride], w2[64 * kTStride], w2t[64 * kTStride], w3[16 * kTStride], w3t[64 * 8];
  __bf16 act[64 * kActStride];   // sample-major: the input, then each layer's activations and errors
  __bf16 x_t[64 * kTStride], h1_t[64 * kTStride], h2_t[64 * kTStride];
  __bf16 d1_t[64 * kTStride], d2_t[64 * kTStride], dz_t[16 * kTStride];
  __bf16 dz_s[64 * 8];
  float z[64 * 8];
  float shift[64], scale[64], b1[64], b2[64], b3[8];
  float red1[4][64], red2[4][64], red3[4][8], red_loss[4][4];
};

// Sum over the 16 lanes of a row, in every lane of it (rotations by 8, 4, 2, 1).
__device__ __forceinline__ float row_sum(float v) {
#define SOMA_ROW_ADD(n)                                                                        \
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + (n), 0xf, 0xf, true))
  SOMA_ROW_ADD(8);
  SOMA_ROW_ADD(4);
  SOMA_ROW_ADD(2);
  SOMA_ROW_ADD(1);
#undef SOMA_ROW_ADD
  return v;
}

// The block's raw features of a chunk: thread t holds quads t + 256 j, quad q =
// features 4 (q mod 16) .. + 3 of sample q / 16 (zero past the batch and past
// feature 59).
struct ChunkFeatures {
  f32x4 v[4];
};

__device__ __forceinline__ ChunkFeatures load_chunk(const TrainArgs &a, uint32_t chunk) {
  ChunkFeatures f;
#pragma unroll
  for (uint32_t j = 0; j < 4u; ++j) {
    const uint32_t q = threadIdx.x + 256u * j, k = 4u * (q & 15u);
    const uint64_t sr = (uint64_t)chunk * 64u + (q >> 4);
    f.v[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (sr < a.n && k < (uint32_t)kNF) f.v[j] = load_f4(a.feat + (size_t)sr * kNF + k, a.vec4);
  }
  return f;
}

// All loads are issued before the first is used: one round trip to memory.
__device__ __forceinline__ void stage_weights(const TrainArgs &a, TrainLds &s) {
  const uint32_t tid = threadIdx.x, o0 = tid >> 4, k = 4u * (tid & 15u);
  f32x4 v1[4], v2[4], v3 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (uint32_t j = 0; j < 4u; ++j) {   // four inputs of output row o0 + 16 j
    const uint32_t o = o0 + 16u * j;
    v1[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (k < (uint32_t)kNF) v1[j] = load_f4(a.params + kPW1 + o * kNF + k, a.vec4);
    v2[j] = load_f4(a.params + kPW2 + o * kNH + k, a.vec4);
  }
  if (o0 < (uint32_t)kNO) v3 = load_f4(a.params + kPW3 + o0 * kNH + k, a.vec4);
  float sh = 0.0f, sc = 0.0f, b1 = 0.0f, b2 = 0.0f, b3 = 0.0f;
  if (tid < 64u) {
    if (tid < (uint32_t)kNF) {
      sh = a.params[kPShift + tid];
      sc = a.params[kPScale + tid];
    }
    b1 = a.params[kPB1 + tid];
    b2 = a.params[kPB2 + tid];
    if (tid < (uint32_t)kNO) b3 = a.params[kPB3 + tid];
  }
#pragma unroll
  for (uint32_t j = 0; j < 4u; ++j) {
    const uint32_t o = o0 + 16u * j;
    *reinterpret_cast<bf16x4 *>(s.w1 + o * kTStride + k) = __builtin_convertvector(v1[j], bf16x4);
    const bf16x4 h = __builtin_convertvector(v2[j], bf16x4);
    *reinterpret_cast<bf16x4 *>(s.w2 + o * kTStride + k) = h;
#pragma unroll
    for (int u = 0; u < 4; ++u) s.w2t[(k + u) * kTStride + o] = h[u];
  }
  const bf16x4 h3 = __builtin_convertvector(v3, bf16x4);
  *reinterpret_cast<bf16x4 *>(s.w3 + o0 * kTStride + k) = h3;
  if (o0 < 8u)
#pragma unroll
    for (int u = 0; u < 4; ++u) s.w3t[(k + u) * 8 + o0] = h3[u];
  if (tid < 64u) {
    s.shift[tid] = sh;
    s.scale[tid] = sc;
    s.b1[tid] = b1;
    s.b2[tid] = b2;
    if (tid < 8u) s.b3[tid] = b3;
  }
  // error rows 6..15 stay zero
  for (uint32_t q = tid; q < 16u * kTStride; q += 256u) s.dz_t[q] = (__bf16)0.0f;
}

// One hidden layer of the wave's 16 samples (row = 16 wv + col of `act`): ReLU
// of the BF16 product plus bias, to the sample's own row and transposed to
// `h_t`; returns the units with a positive input, bit 4 mt + r.
__device__ __forceinline__ uint32_t train_layer(const __bf16 *w, const float *bias, __bf16 *act,
                                                __bf16 *h_t, uint32_t wv) {
  const uint32_t lane = threadIdx.x & 63u, col = lane & 15u, g = lane >> 4, sm = 16u * wv + col;
  bf16x8 b[2];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) b[kb] = lds8(act + sm * kActStride + 32 * kb + 8 * g);
  wave_lds_fence();
  uint32_t on = 0u;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds8(w + (16 * mt + col) * kTStride + 32 * kb + 8 * g),
                                                    b[kb], acc, 0, 0, 0);
    const uint32_t u = 16u * mt + 4u * g;
    const f32x4 pre = acc + *reinterpret_cast<const f32x4 *>(bias + u);
    bf16x4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h[r] = (__bf16)relu(pre[r]);
      on |= pre[r] > 0.0f ? 1u << (4 * mt + r) : 0u;
    }
    *reinterpret_cast<bf16x4 *>(act + sm * kActStride + u) = h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h_t[(u + r) * kTStride + sm] = h[r];
  }
  wave_lds_fence();
  return on;
}

// One block per partial gradient, four waves.  Bound by latency (a chain of six
// small products per chunk and the traffic through LDS between them), which is
// why a chunk is spread over four waves, all loads of a chunk and of the weights
// are in flight together, and the weights are converted here instead of by a
// kernel before it.  Batch 8192 (128 chunks), whole step: 15.9 us (11.4 us here,
// of which a third is one round trip to memory); 46.7 us with one wave per chunk,
// strided feature loads and three launches.
__global__ __launch_bounds__(256) void mlp_grad_kernel(const TrainArgs a) {
  __shared__ TrainLds s;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6, col = lane & 15u, g = lane >> 4;
  const uint32_t sm = 16u * wv + col;   // the lane's sample within the chunk
  ChunkFeatures next = load_chunk(a, blockIdx.x);   // in flight while the weights are staged
  stage_weights(a, s);
  f32x4 gw1[4], gw2[4], gw3 = {0.f, 0.f, 0.f, 0.f}, gb1[4], gb2[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) gw1[i] = gw2[i] = gb1[i] = gb2[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gmu = 0.0f, gls = 0.0f, loss = 0.0f;   // output-bias gradients of dimension g

  const uint32_t n_chunks = (a.n + 63u) / 64u;
  for (uint32_t chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x) {
    const uint32_t s0 = chunk * 64u;
    __syncthreads();   // the tiles of the chunk before are read; the weights are staged
    // standardised inputs, sample-major and unit-major
#pragma unroll
    for (uint32_t j = 0; j < 4u; ++j) {
      const uint32_t q = tid + 256u * j, sr = q >> 4, k = 4u * (q & 15u);
      const f32x4 v = (next.v[j] - *reinterpret_cast<const f32x4 *>(s.shift + k)) *
                      *reinterpret_cast<const f32x4 *>(s.scale + k);
      const bf16x4 h = __builtin_convertvector(v, bf16x4);
      *reinterpret_cast<bf16x4 *>(s.act + sr * kActStride + k) = h;
#pragma unroll
      for (int u = 0; u < 4; ++u) s.x_t[(k + u) * kTStride + sr] = h[u];
    }
    if (chunk + gridDim.x < n_chunks) next = load_chunk(a, chunk + gridDim.x);
    __syncthreads();
    const uint32_t on1 = train_layer(s.w1, s.b1, s.act, s.h1_t, wv);
    const uint32_t on2 = train_layer(s.w2, s.b2, s.act, s.h2_t, wv);
    {   // output layer: rows 0..5 of one tile
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds8(s.w3 + col * kTStride + 32 * kb + 8 * g),
                                                      lds8(s.act + sm * kActStride + 32 * kb + 8 * g),
                                                      acc, 0, 0, 0);
      if (g < 2u) *reinterpret_cast<f32x4 *>(s.z + sm * 8 + 4 * g) =
          acc + *reinterpret_cast<const f32x4 *>(s.b3 + 4 * g);
    }
    wave_lds_fence();
    // loss and dL/dz: lane row g takes dimension g of the lane's sample
    {
      const uint32_t d = g < 3u ? g : 0u;
      const bool valid = g < 3u && s0 + sm < a.n;
      const float tgt = valid ? a.target[(size_t)(s0 + sm) * 3u + d] : 0.0f;
      const float mu = a.head.m_max * tanhf(s.z[sm * 8 + d] / a.head.m_max);
      const float sg = fast_rcp(1.0f + __expf(-s.z[sm * 8 + 3 + d]));
      const float ls = a.head.lo + (a.head.hi - a.head.lo) * sg;
      const float inv_var = __expf(-2.0f * ls);
      const float e = tgt - mu;
      if (valid) loss += 0.5f * e * e * inv_var + ls;
      const float dmu = -e * inv_var, dls = 1.0f - e * e * inv_var;
      const float zm = valid ? dmu * (1.0f - (mu / a.head.m_max) * (mu / a.head.m_max)) : 0.0f;
      const float zl = valid ? dls * (a.head.hi - a.head.lo) * sg * (1.0f - sg) : 0.0f;
      gmu += zm;
      gls += zl;
      if (g < 3u) {
        const __bf16 bm = (__bf16)zm, bl = (__bf16)zl;
        s.dz_s[sm * 8 + d] = bm;
        s.dz_s[sm * 8 + 3 + d] = bl;
        s.dz_t[d * kTStride + sm] = bm;
        s.dz_t[(3 + d) * kTStride + sm] = bl;
      } else {
        s.dz_s[sm * 8 + 6] = s.dz_s[sm * 8 + 7] = (__bf16)0.0f;
      }
    }
    wave_lds_fence();
    // delta2 = (W3^T dz) * relu'(a2): K = 32 with outputs 0..7 in lane row 0
    const bf16x8 zero8 = {};
    const bf16x8 bz = g == 0u ? lds8(s.dz_s + sm * 8) : zero8;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 av = g == 0u ? lds8(s.w3t + (16 * mt + col) * 8) : zero8;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bz, acc, 0, 0, 0);
      const uint32_t u = 16u * mt + 4u * g;
      f32x4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) d[r] = acc[r] * ((on2 >> (4 * mt + r)) & 1u ? 1.0f : 0.0f);
      gb2[mt] += d;
      const bf16x4 db = __builtin_convertvector(d, bf16x4);
      *reinterpret_cast<bf16x4 *>(s.act + sm * kActStride + u) = db;
#pragma unroll
      for (int r = 0; r < 4; ++r) s.d2_t[(u + r) * kTStride + sm] = db[r];
    }
    wave_lds_fence();
    // delta1 = (W2^T delta2) * relu'(a1)
    bf16x8 b2[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) b2[kb] = lds8(s.act + sm * kActStride + 32 * kb + 8 * g);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            lds8(s.w2t + (16 * mt + col) * kTStride + 32 * kb + 8 * g), b2[kb], acc, 0, 0, 0);
      const uint32_t u = 16u * mt + 4u * g;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float d = acc[r] * ((on1 >> (4 * mt + r)) & 1u ? 1.0f : 0.0f);
        gb1[mt][r] += d;
        s.d1_t[(u + r) * kTStride + sm] = (__bf16)d;
      }
    }
    __syncthreads();
    // weight gradients, contracted over the chunk's samples: input units 16 wv + col
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const uint32_t at = 32u * kb + 8u * g;
      const bf16x8 bx = lds8(s.x_t + sm * kTStride + at), bh1 = lds8(s.h1_t + sm * kTStride + at),
                   bh2 = lds8(s.h2_t + sm * kTStride + at);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        gw1[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds8(s.d1_t + (16 * mt + col) * kTStride + at),
                                                          bx, gw1[mt], 0, 0, 0);
        gw2[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds8(s.d2_t + (16 * mt + col) * kTStride + at),
                                                          bh1, gw2[mt], 0, 0, 0);
      }
      gw3 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lds8(s.dz_t + col * kTStride + at), bh2, gw3, 0, 0, 0);
    }
  }

  // the block's partial gradient in the parameter layout
  float *out = a.partials + (size_t)blockIdx.x * kPSize;
  const uint32_t i = 16u * wv + col;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t o = 16u * mt + 4u * g + r;
      if (i < (uint32_t)kNF) out[kPW1 + o * kNF + i] = gw1[mt][r];
      out[kPW2 + o * kNH + i] = gw2[mt][r];
      if (mt == 0 && o < (uint32_t)kNO) out[kPW3 + o * kNH + i] = gw3[r];
    }
  // bias and loss partials: over the 16 samples of a wave, then over the waves in order
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v1 = row_sum(gb1[mt][r]), v2 = row_sum(gb2[mt][r]);
      if (col == 0u) {
        s.red1[wv][16 * mt + 4 * g + r] = v1;
        s.red2[wv][16 * mt + 4 * g + r] = v2;
      }
    }
  gmu = row_sum(gmu);
  gls = row_sum(gls);
  loss = row_sum(loss);
  if (col == 0u) {
    if (g < 3u) {
      s.red3[wv][g] = gmu;
      s.red3[wv][3 + g] = gls;
    }
    s.red_loss[wv][g] = loss;
  }
  __syncthreads();
  if (tid < 64u) {
    out[kPB1 + tid] = (s.red1[0][tid] + s.red1[1][tid]) + (s.red1[2][tid] + s.red1[3][tid]);
    out[kPB2 + tid] = (s.red2[0][tid] + s.red2[1][tid]) + (s.red2[2][tid] + s.red2[3][tid]);
    if (tid < (uint32_t)kNO)
      out[kPB3 + tid] = (s.red3[0][tid] + s.red3[1][tid]) + (s.red3[2][tid] + s.red3[3][tid]);
    const float l = row_sum(s.red_loss[(tid >> 2) & 3u][tid & 3u]);   // 16 values, lanes 0..15
    if (tid == 0u) a.loss_partials[blockIdx.x] = l;
  }
  if (tid < (uint32_t)kPW1) out[tid] = 0.0f;   // no gradient for the standardisation
  if (tid < (uint32_t)(kPSize - kPB3 - kNO)) out[kPB3 + kNO + tid] = 0.0f;
}

struct AdamArgs {
  const float *partials;
  const float *loss_partials;
  uint32_t waves, n;
  float *params, *m, *v;
  float lr, beta1, beta2, eps;
  float bc1, bc2;        // 1 - beta^t
  int apply;
  float *grad_out;       // may be null
  float *loss_out;       // may be null
};

// Mean gradient over the batch and the Adam step on the FP32 master
// parameters (standardisation constants untouched).  A block covers 64
// parameters; its 16 waves sum the partials of blocks q, q+16, q+32, ... (q the
// wave in the block), eight loads in flight, and the 16 sums are combined in a
// fixed order: the result does not depend on timing.  Bound by the latency of
// its loads: 128 partials are one round of eight loads per wave (four rounds
// with four waves, and a serial sum of the losses, took 9.2 us).
constexpr uint32_t kAdamParamsPerBlock = 64;
constexpr uint32_t kAdamWaves = 16;

__global__ __launch_bounds__(64 * kAdamWaves) void mlp_adam_kernel(const AdamArgs a) {
  __shared__ float s_part[kAdamWaves][kAdamParamsPerBlock];
  const uint32_t lane = threadIdx.x & 63u, q = threadIdx.x >> 6;
  const uint32_t p = blockIdx.x * kAdamParamsPerBlock + lane;
  float gsum = 0.0f;
  if (p < (uint32_t)kPSize) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (uint32_t w = q; w < a.waves; w += 8u * kAdamWaves) {
#pragma unroll
      for (uint32_t u = 0; u < 8u; ++u) {
        const uint32_t ww = w + kAdamWaves * u;
        if (ww < a.waves) acc[u] += a.partials[(size_t)ww * kPSize + p];
      }
    }
    gsum = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  }
  s_part[q][lane] = gsum;
  __syncthreads();
  if (blockIdx.x == 0 && q == 1u && a.loss_out) {
    float l = 0.0f;
    for (uint32_t w = lane; w < a.waves; w += 64u) l += a.loss_partials[w];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0u) *a.loss_out = l / (float)a.n;
  }
  if (q != 0 || p >= (uint32_t)kPSize) return;
  float part[kAdamWaves];
#pragma unroll
  for (uint32_t w = 0; w < kAdamWaves; ++w) part[w] = s_part[w][lane];
#pragma unroll
  for (uint32_t half = kAdamWaves / 2u; half > 0u; half >>= 1)
#pragma unroll
    for (uint32_t w = 0; w < half; ++w) part[w] += part[w + half];
  const float grad = part[0] / (float)a.n;
  if (a.grad_out) a.grad_out[p] = grad;
  if (!a.apply || p < (uint32_t)kPW1 || p >= (uint32_t)(kPB3 + kNO)) return;
  const float m = a.beta1 * a.m[p] + (1.0f - a.beta1) * grad;
  const float v = a.beta2 * a.v[p] + (1.0f - a.beta2) * grad * grad;
  a.m[p] = m;
  a.v[p] = v;
  a.params[p] -= a.lr * (m / a.bc1) / (sqrtf(v / a.bc2) + a.eps);
}

}  // namespace soma
