// Decoder MLP 32 -> 64 -> 64 -> 4 (Sec. 3.1, Eq. 1-2: the shallow MLP that
// turns concatenated hash features into density and colour) on MFMA.
//
// Layer products are out[m][n] = sum_k W[m][k] in[k][n] with m = neuron,
// n = sample (16 per tile), k = input.  One wave owns a 16-sample tile.
// MFMA operand layouts (lane l, r = l % 16, g = l / 16):
//   v_mfma_f32_16x16x4_f32   : A[r][g], B[g][r] (one value each), D[4g+i][r]
//   v_mfma_f32_16x16x32_bf16 : A[r][8g+j], B[8g+j][r] (8 bf16 each), D[4g+i][r]
// A lane therefore ends a layer holding neurons {16t + 4g + i} of sample r.
// The next layer consumes exactly those registers as its B operand by
// ordering its K dimension the same way (k-step (t, i), slot g = neuron
// 16t + 4g + i); its weight fragments are gathered in that order.  So the
// activations never leave registers between layers.  Features arrive
// level-major [L][S][2]: lane group g reads levels 4g..4g+3 of its sample,
// i.e. features 8g..8g+7, which fixes the K order of the first layer.
#include <hip/hip_bf16.h>

#include "common.h"
#include "mlp_dev.h"

using namespace ia355;
using namespace ia355::mlpd;

namespace {

constexpr int kMlpBlock = 256;

// LDS copy of the parameters, rows padded so that the lanes (r, g) of a
// fragment read distinct banks along rows and along columns
constexpr int PW1 = 36, PW2 = 68, PW3 = 80;
constexpr int PO_W1 = 0, PO_W2 = PO_W1 + NH * PW1, PO_W3 = PO_W2 + NH * PW2, PO_B1 = PO_W3 + NOUT * PW3,
              PO_B2 = PO_B1 + NH, PO_B3 = PO_B2 + NH, PO_SIZE = PO_B3 + NOUT;
__device__ __forceinline__ void stage_padded(const float *__restrict__ P, float *p) {
  const float4 *P4 = reinterpret_cast<const float4 *>(P);
  constexpr int kPer = (NPARAM / 4 + kMlpBlock - 1) / kMlpBlock, kLast = NPARAM / 4 - 1;
  float4 v[kPer];
  // every load in flight before the first is used; threads past the end copy
  // the last group again
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * kMlpBlock;
    v[k] = P4[e < kLast ? e : kLast];
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) asm volatile("" : "+v"(v[k].x), "+v"(v[k].y), "+v"(v[k].z), "+v"(v[k].w));
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * kMlpBlock, i = 4 * (e < kLast ? e : kLast);
    int o = PO_B3 + i - OFF_B3;
    o = i < OFF_B3 ? PO_W3 + ((i - OFF_W3) / NH) * PW3 + (i - OFF_W3) % NH : o;
    o = i < OFF_W3 ? PO_B2 + i - OFF_B2 : o;
    o = i < OFF_B2 ? PO_W2 + ((i - OFF_W2) / NH) * PW2 + (i - OFF_W2) % NH : o;
    o = i < OFF_W2 ? PO_B1 + i - OFF_B1 : o;
    o = i < OFF_B1 ? PO_W1 + (i / NIN) * PW1 + i % NIN : o;
    *reinterpret_cast<float4 *>(p + o) = v[k];
  }
}

__device__ __forceinline__ f32x4 splat(float v) { return f32x4{v, v, v, v}; }

// acc + the products of four k-steps.
__device__ __forceinline__ f32x4 mfma4x4(const f32x4 &a, const f32x4 &b, f32x4 acc) {
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = mfma4(a[i], b[i], acc);
  return acc;
}

__device__ __forceinline__ f32x4 relu4(const f32x4 &z) {
  return f32x4{relu(z[0]), relu(z[1]), relu(z[2]), relu(z[3])};
}

// The activated output of lane (r, g), output g of sample r, given as its
// pre-activation o: the density exp(o) (clamped at exp(80)) or a colour
// sigmoid(o), as head() computes them.
__device__ __forceinline__ float head_lane(int g, float o) {
  const float e = expf(g == 0 ? fminf(o, 80.0f) : -o);
  return g == 0 ? e : __builtin_amdgcn_rcpf(1.0f + e);
}

// --------------------------------------------------------------- forward
// A wave takes 16 samples at a time, the inputs of the next kFwdPre tiles in
// flight (a tile's MFMA chain is far shorter than a load's latency).  The last
// layer's operand has W3's rows at 0, 4, 8 and 12 and zeros between, so lane
// (r, g) ends with output g of sample r: one exponential and one store a lane.
constexpr int kFwdPre = 2;

// The inputs of a 16-sample tile for lane (r, g): loaded for a valid sample
// index in any case, so that nothing branches around the loads.
struct F32X {
  float2 x[4];  // levels 4g .. 4g + 3 of sample r
  int16_t bone;
};

template <bool kBone>
__device__ __forceinline__ void load_x(const float2 *feat, const int16_t *bone, int64_t S, int64_t ld,
                                       int64_t s, int g, F32X &in) {
  s = s < S ? s : S - 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) in.x[j] = feat[(int64_t)(4 * g + j) * ld + s];
  in.bone = kBone ? bone[s] : (int16_t)0;
}

// FP32: the two hidden layers' weights in registers (two waves per SIMD).
// 36,503 samples: 11 us, 262,144: 36.  With fragments gathered one
// conflicting LDS word at a time and sixteen lanes computing the four outputs
// of their samples: 12.5 and 41.6 us.
template <bool kBone>
__global__ void __launch_bounds__(kMlpBlock, 2) mlp_fwd_f32(const float *__restrict__ feat,
                                                            const int16_t *__restrict__ bone, int64_t S,
                                                            const int64_t *__restrict__ S_dev, int64_t ld,
                                                            const float *__restrict__ P, float *__restrict__ sigma,
                                                            float *__restrict__ rgb) {
  __shared__ __attribute__((aligned(16))) float p[PO_SIZE];
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  S = count_of(S, S_dev);
  const int64_t ntile = ceil_div(S, 16), wstride = (int64_t)gridDim.x * (kMlpBlock / 64);
  int64_t tile = (int64_t)blockIdx.x * (kMlpBlock / 64) + wid;
  if ((int64_t)blockIdx.x * (kMlpBlock / 64) >= ntile) return;  // the whole block (before the barrier)
  const float2 *feat2 = reinterpret_cast<const float2 *>(feat);
  F32X in[kFwdPre];
#pragma unroll
  for (int u = 0; u < kFwdPre; ++u) load_x<kBone>(feat2, bone, S, ld, (tile + u * wstride) * 16 + r, g, in[u]);
  stage_padded(P, p);
  __syncthreads();
  f32x4 w1[4][2], w2[4][4], w3[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int c = 0; c < 2; ++c) w1[mt][c] = *reinterpret_cast<const f32x4 *>(p + PO_W1 + (16 * mt + r) * PW1 + 8 * g + 4 * c);
#pragma unroll
    for (int t = 0; t < 4; ++t) w2[mt][t] = *reinterpret_cast<const f32x4 *>(p + PO_W2 + (16 * mt + r) * PW2 + 16 * t + 4 * g);
    const f32x4 v = *reinterpret_cast<const f32x4 *>(p + PO_W3 + (r >> 2) * PW3 + 16 * mt + 4 * g);
    w3[mt] = (r & 3) == 0 ? v : splat(0.0f);
  }
  const float b3 = p[PO_B3 + g];
  float *out = g == 0 ? sigma : rgb + (g - 1) * ld;
  for (; tile < ntile; tile += kFwdPre * wstride) {
#pragma unroll
    for (int u = 0; u < kFwdPre; ++u) {
      if (tile + u * wstride >= ntile) break;
      const int64_t s = (tile + u * wstride) * 16 + r;
      const bool ok = s < S;
      f32x4 X[2];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        X[j / 2][2 * (j % 2)] = in[u].x[j].x;
        X[j / 2][2 * (j % 2) + 1] = in[u].x[j].y;
      }
      const bool use = !kBone || in[u].bone >= 0;
      f32x4 z[4], h[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        z[mt] = *reinterpret_cast<const f32x4 *>(p + PO_B1 + 16 * mt + 4 * g);
#pragma unroll
        for (int c = 0; c < 2; ++c) z[mt] = mfma4x4(w1[mt][c], X[c], z[mt]);
        h[mt] = relu4(z[mt]);
      }
      // only now, into the registers that the first layer has read
      __builtin_amdgcn_sched_barrier(0);
      load_x<kBone>(feat2, bone, S, ld, s + kFwdPre * wstride * 16, g, in[u]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        z[mt] = *reinterpret_cast<const f32x4 *>(p + PO_B2 + 16 * mt + 4 * g);
#pragma unroll
        for (int t = 0; t < 4; ++t) z[mt] = mfma4x4(w2[mt][t], h[t], z[mt]);
      }
      f32x4 o = {b3, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int t = 0; t < 4; ++t) o = mfma4x4(w3[t], relu4(z[t]), o);
      const float v = head_lane(g, o[0]);
      if (ok) out[s] = use ? v : 0.0f;
    }
  }
}

// BF16: the weights in LDS, read as the MFMAs need them (held in registers
// they cost 90 a lane, two waves per SIMD), each read serving kBfTiles tiles:
// with one, the 22 16-byte reads of a tile took two thirds of the time.
// 1,000,003 samples: 24 us (one tile a read: 27); with branches around the
// loads, serial waits in the weights' staging and sixteen lanes computing the
// four outputs of their samples 35 us.
constexpr int kBfTiles = 2;

struct BfX {
  uint32_t x[4];  // levels 4g .. 4g + 3 of sample r
  int16_t bone;
};

template <bool kBone>
__device__ __forceinline__ void load_x(const uint32_t *feat, const int16_t *bone, int64_t S, int64_t ld, int64_t s,
                                       int g, BfX &in) {
  s = s < S ? s : S - 1;
#pragma unroll
  for (int j = 0; j < 4; ++j) in.x[j] = feat[(int64_t)(4 * g + j) * ld + s];
  in.bone = kBone ? bone[s] : (int16_t)0;
}

// A whole block fills the store from the parameters in global memory (16-byte
// aligned), each fragment two 16-byte loads of consecutive parameters,
// converted as frag_value converts them; W3's rows go to 0, 4, 8 and 12.
// Every load is in flight before the first is used.
__device__ __forceinline__ void stage_frag_spread(const float *__restrict__ P, FragLds &s) {
  constexpr int kPer = (14 * 64 + kMlpBlock - 1) / kMlpBlock;
  float4 v[kPer][2];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * kMlpBlock, q = e < 14 * 64 ? e >> 6 : 13, r = e & 15, g = (e >> 4) & 3;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      v[k][h] = *reinterpret_cast<const float4 *>(P + frag_half_at(q, q < 12 ? r : r >> 2, g, h));
  }
  const int b = threadIdx.x < 2 * NH ? (threadIdx.x < NH ? OFF_B1 : OFF_B2 - NH) + threadIdx.x
                                     : OFF_B3 + (threadIdx.x & (NOUT - 1));
  float bias = P[b];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      asm volatile("" : "+v"(v[k][h].x), "+v"(v[k][h].y), "+v"(v[k][h].z), "+v"(v[k][h].w));
  asm volatile("" : "+v"(bias));
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = threadIdx.x + k * kMlpBlock, q = e >> 6;
    if (e >= 14 * 64) break;
    bf16x8 f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f[4 * h] = (__bf16)v[k][h].x;
      f[4 * h + 1] = (__bf16)v[k][h].y;
      f[4 * h + 2] = (__bf16)v[k][h].z;
      f[4 * h + 3] = (__bf16)v[k][h].w;
    }
    const bf16x8 zero = {};
    s.mw[q][e & 63] = q < 12 || (e & 3) == 0 ? f : zero;
  }
  if (threadIdx.x < 2 * NH)
    (threadIdx.x < NH ? s.b1 : s.b2 - NH)[threadIdx.x] = bias;
  else if (threadIdx.x < 2 * NH + NOUT)
    s.b3[threadIdx.x - 2 * NH] = bias;
}

template <bool kBone>
__global__ void __launch_bounds__(kMlpBlock, 4) mlp_fwd_bf16(const __hip_bfloat16 *__restrict__ featb,
                                                            const int16_t *__restrict__ bone, int64_t S,
                                                            const int64_t *__restrict__ S_dev, int64_t ld,
                                                            const float *__restrict__ P, float *__restrict__ sigma,
                                                            float *__restrict__ rgb) {
  __shared__ __attribute__((aligned(16))) FragLds sF;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  S = count_of(S, S_dev);
  const int64_t nstep = ceil_div(S, 16 * kBfTiles), wstride = (int64_t)gridDim.x * (kMlpBlock / 64);
  int64_t st = (int64_t)blockIdx.x * (kMlpBlock / 64) + wid;
  if ((int64_t)blockIdx.x * (kMlpBlock / 64) >= nstep) return;  // the whole block (before the barrier)
  const uint32_t *feat = reinterpret_cast<const uint32_t *>(featb);
  BfX in[kBfTiles];
#pragma unroll
  for (int u = 0; u < kBfTiles; ++u) load_x<kBone>(feat, bone, S, ld, (st * kBfTiles + u) * 16 + r, g, in[u]);
  stage_frag_spread(P, sF);
  __syncthreads();
  const LdsW w{sF, lane, g};
  const float b3 = sF.b3[g];
  float *out = g == 0 ? sigma : rgb + (g - 1) * ld;
  for (; st < nstep; st += wstride) {
    bf16x8 X[kBfTiles], ha[kBfTiles], hb[kBfTiles];
    bool use[kBfTiles];
#pragma unroll
    for (int u = 0; u < kBfTiles; ++u) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        X[u][2 * j] = __builtin_bit_cast(__bf16, (uint16_t)(in[u].x[j] & 0xffffu));
        X[u][2 * j + 1] = __builtin_bit_cast(__bf16, (uint16_t)(in[u].x[j] >> 16));
      }
      use[u] = !kBone || in[u].bone >= 0;
    }
    pin_in_loop();
    f32x4 z[kBfTiles][4], o[kBfTiles];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 a = w.w1(mt);
      const f32x4 b = w.b1(mt);
#pragma unroll
      for (int u = 0; u < kBfTiles; ++u) z[u][mt] = mfma32(a, X[u], b);
    }
    // only now, into the registers that the first layer has read
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < kBfTiles; ++u) {
      load_x<kBone>(feat, bone, S, ld, ((st + wstride) * kBfTiles + u) * 16 + r, g, in[u]);
      ha[u] = pack_act(z[u], 0);
      hb[u] = pack_act(z[u], 1);
      o[u] = f32x4{b3, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 a0 = w.w2(mt, 0), a1 = w.w2(mt, 1);
      const f32x4 b = w.b2(mt);
#pragma unroll
      for (int u = 0; u < kBfTiles; ++u) z[u][mt] = mfma32(a1, hb[u], mfma32(a0, ha[u], b));
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const bf16x8 a = w.w3(c);
#pragma unroll
      for (int u = 0; u < kBfTiles; ++u) o[u] = mfma32(a, pack_act(z[u], c), o[u]);
    }
#pragma unroll
    for (int u = 0; u < kBfTiles; ++u) {
      const int64_t s = (st * kBfTiles + u) * 16 + r;
      const float v = head_lane(g, o[u][0]);
      if (s < S) out[s] = use[u] ? v : 0.0f;
    }
  }
}

// --------------------------------------------------------------- backward
// Per sample: recompute the forward, then
//   d3 = dL/do (exp / sigmoid heads), gh2 = W3^T d3, d2 = gh2 * [z2 >= 0],
//   gh1 = W2^T d2, d1 = gh1 * [z1 >= 0], gfeat = W1^T d1,
//   dW3 += d3 h2^T, dW2 += d2 h1^T, dW1 += d1 x^T, db += sum d.
// The transposed products chain in registers like the forward.  Each of a
// workgroup's four waves takes 16 of its 64 samples through the forward and
// the deltas; then the waves share the weight gradients, wave w the rows of
// neurons 16w .. 16w + 15, with K = the 64 samples from [neuron][sample] tiles
// in LDS.  So a wave holds 28 accumulator registers, not 112, and works
// without moves to and from the accumulation registers.  The next step's
// inputs are in flight during a step.  Block partials are reduced in a fixed
// order.
constexpr int kBwdBlock = kMlpBlock, kBwdWaves = kBwdBlock / 64;
constexpr int kBwdSamples = 16 * kBwdWaves;  // per block and step
// rows of the sample tiles
constexpr int BR_X = 0, BR_H1 = 32, BR_H2 = 96, BR_D2 = 160, BR_D1 = 224, BR_D3 = 288, BR_ROWS = 292;
// --------------------------------------------------------------- FP32 bwd
// Bound by the FP32 matrix rate: 324 MFMAs of 32 cycles for 16 samples.
// 36,503 samples: 28 us.  Two waves a block with every accumulator, waiting
// for each tile's loads, took 48 us: 8 of preparing weights, 9.7 us per 16
// samples and 8 of adding the waves.
constexpr int LDF = kBwdSamples + 4;  // row stride of the sample tiles
struct F32BwdLds {
  union {
    float p[PO_SIZE];
    float t[BR_ROWS * LDF];
  };
  // fragments of four k-steps: 4 mt + t of W2's transpose, 16 + 4 mt + t of
  // W1's, 24 + t of W3
  f32x4 w[28][64];
  float b1[NH], b2[NH];
};
static_assert(sizeof(F32BwdLds) <= 160 * 1024, "one workgroup's LDS");

struct F32In {
  F32X x;
  float go;  // gradient of output g of sample r
};

template <bool kBone>
__device__ __forceinline__ void load_in(const float2 *feat, const float *go, const int16_t *bone, int64_t S,
                                        int64_t ld, int64_t s, int g, F32In &in) {
  load_x<kBone>(feat, bone, S, ld, s, g, in.x);
  in.go = go[s < S ? s : S - 1];
}

template <bool kBone>
__global__ void __launch_bounds__(kBwdBlock, 2) mlp_bwd_f32(const float *__restrict__ gsig,
                                                            const float *__restrict__ grgb,
                                                            const float *__restrict__ feat,
                                                            const int16_t *__restrict__ bone, int64_t S,
                                                            const int64_t *__restrict__ S_dev, int64_t ld,
                                                            const float *__restrict__ P, float *__restrict__ gfeat,
                                                            float *__restrict__ partial) {
  extern __shared__ __attribute__((aligned(16))) unsigned char f32_lds[];
  F32BwdLds &lds = *reinterpret_cast<F32BwdLds *>(f32_lds);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const float2 *feat2 = reinterpret_cast<const float2 *>(feat);
  S = count_of(S, S_dev);
  const int64_t step = (int64_t)gridDim.x * kBwdSamples;
  const float *go = g == 0 ? gsig : grgb + (g - 1) * ld;
  int64_t s0 = (int64_t)blockIdx.x * kBwdSamples + 16 * wid;
  F32In in = {};
  if (S > 0) load_in<kBone>(feat2, go, bone, S, ld, s0 + r, g, in);
  stage_padded(P, lds.p);
  __syncthreads();
  const float *p = lds.p;
  f32x4 w1[4][2], w2[4][4];
  float w3t[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int c = 0; c < 2; ++c) w1[mt][c] = *reinterpret_cast<const f32x4 *>(p + PO_W1 + (16 * mt + r) * PW1 + 8 * g + 4 * c);
#pragma unroll
    for (int t = 0; t < 4; ++t) w2[mt][t] = *reinterpret_cast<const f32x4 *>(p + PO_W2 + (16 * mt + r) * PW2 + 16 * t + 4 * g);
    w3t[mt] = p[PO_W3 + g * PW3 + 16 * mt + r];
  }
  const float b3 = p[PO_B3 + g];
  // the fragments in LDS, a quarter by each wave: [16t + 4g + i][16mt + r] of
  // W2, W1; W3[r / 4][16t + 4g + i] in the rows r = 0, 4, .. and zero in the
  // others, so that lane (r, g) gets output g of sample r
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const int q = kBwdWaves * k + wid, mt = (q & 15) >> 2, t = q & 3;
    f32x4 v;
    if (k < 6) {
      const float *col = p + (k < 4 ? PO_W2 : PO_W1) + 16 * mt + r;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = col[(16 * t + 4 * g + i) * (k < 4 ? PW2 : PW1)];
    } else {
      v = *reinterpret_cast<const f32x4 *>(p + PO_W3 + (r >> 2) * PW3 + 16 * t + 4 * g);
      v = (r & 3) == 0 ? v : splat(0.0f);
    }
    lds.w[q][lane] = v;
  }
  if (threadIdx.x < 2 * NH) (threadIdx.x < NH ? lds.b1 : lds.b2 - NH)[threadIdx.x] = p[PO_B1 + threadIdx.x];
  __syncthreads();  // the tiles take the parameters' place
  f32x4 aW1[2], aW2[4], aW3 = splat(0.0f);
  float ab1 = 0.0f, ab2 = 0.0f, ab3 = 0.0f;  // of neuron 16 wid + r, output r
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    aW2[a] = splat(0.0f);
    if (a < 2) aW1[a] = splat(0.0f);
  }
  float *tc = lds.t + 16 * wid + r;  // this lane's sample in row 0
  for (int64_t c0 = (int64_t)blockIdx.x * kBwdSamples; c0 < S; c0 += step, s0 += step) {  // uniform in the block
    const int64_t s = s0 + r;
    const bool ok = s < S, use = ok && (!kBone || in.x.bone >= 0);
    f32x4 X[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      X[j / 2][2 * (j % 2)] = ok ? in.x.x[j].x : 0.0f;
      X[j / 2][2 * (j % 2) + 1] = ok ? in.x.x[j].y : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) tc[(BR_X + 8 * g + k) * LDF] = X[k / 4][k % 4];
    const float go_s = in.go;
    // the next step's inputs (after the last: the last sample's again)
    load_in<kBone>(feat2, go, bone, S, ld, s + step, g, in);
    f32x4 z1[4], z2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      z1[mt] = *reinterpret_cast<const f32x4 *>(lds.b1 + 16 * mt + 4 * g);
#pragma unroll
      for (int c = 0; c < 2; ++c) z1[mt] = mfma4x4(w1[mt][c], X[c], z1[mt]);
    }
    f32x4 h[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      h[t] = relu4(z1[t]);
#pragma unroll
      for (int i = 0; i < 4; ++i) tc[(BR_H1 + 16 * t + 4 * g + i) * LDF] = h[t][i];
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      z2[mt] = *reinterpret_cast<const f32x4 *>(lds.b2 + 16 * mt + 4 * g);
#pragma unroll
      for (int t = 0; t < 4; ++t) z2[mt] = mfma4x4(w2[mt][t], h[t], z2[mt]);
    }
    f32x4 oa = {b3, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      h[t] = relu4(z2[t]);
#pragma unroll
      for (int i = 0; i < 4; ++i) tc[(BR_H2 + 16 * t + 4 * g + i) * LDF] = h[t][i];
      oa = mfma4x4(lds.w[24 + t][lane], h[t], oa);
    }
    // the gradient of output g of sample r
    const float o = oa[0], e = expf(g == 0 ? fminf(o, 80.0f) : -o), c = __builtin_amdgcn_rcpf(1.0f + e);
    float d3 = g == 0 ? (o < 80.0f ? go_s * e : 0.0f) : go_s * c * (1.0f - c);
    d3 = use ? d3 : 0.0f;
    tc[(BR_D3 + g) * LDF] = d3;
    f32x4 d2[4], d1[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      d2[mt] = mfma4(w3t[mt], d3, splat(0.0f));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d2[mt][i] = z2[mt][i] < 0.0f ? 0.0f : d2[mt][i];
        tc[(BR_D2 + 16 * mt + 4 * g + i) * LDF] = d2[mt][i];
      }
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      d1[mt] = splat(0.0f);
#pragma unroll
      for (int t = 0; t < 4; ++t) d1[mt] = mfma4x4(lds.w[4 * mt + t][lane], d2[t], d1[mt]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d1[mt][i] = z1[mt][i] < 0.0f ? 0.0f : d1[mt][i];
        tc[(BR_D1 + 16 * mt + 4 * g + i) * LDF] = d1[mt][i];
      }
    }
    // gfeat = W1^T d1 -> feature 16mt + 4g + i = level 8mt + 2g + i/2, f = i%2
    if (gfeat) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        f32x4 acc = splat(0.0f);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc = mfma4x4(lds.w[16 + 4 * mt + t][lane], d1[t], acc);
        if (ok) {
          float2 *gf = reinterpret_cast<float2 *>(gfeat);
          gf[(int64_t)(8 * mt + 2 * g) * ld + s] = make_float2(acc[0], acc[1]);
          gf[(int64_t)(8 * mt + 2 * g + 1) * ld + s] = make_float2(acc[2], acc[3]);
        }
      }
    }
    __syncthreads();
    // weight gradients of this wave's rows, K = the block's samples (slot g of
    // step i: sample 16k + 4g + i), each 32 samples summed from zero, then the
    // two sums, so that the chains of roundings stay short
    const float *tr = lds.t + r * LDF + 4 * g;
    auto rows = [&](int row, int k) { return *reinterpret_cast<const f32x4 *>(tr + row * LDF + 16 * k); };
    auto products = [&](const f32x4 v[4], int row) {
      const f32x4 a = mfma4x4(v[1], rows(row, 1), mfma4x4(v[0], rows(row, 0), splat(0.0f)));
      return a + mfma4x4(v[3], rows(row, 3), mfma4x4(v[2], rows(row, 2), splat(0.0f)));
    };
    auto sum = [](const f32x4 v[4]) {
      float s[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]);
      return (s[0] + s[1]) + (s[2] + s[3]);
    };
    static_assert(kBwdSamples == 64, "four sets of 16 samples");
    f32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = rows(BR_D2 + 16 * wid, k);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) aW2[nt] += products(v, BR_H1 + 16 * nt);
    ab2 += sum(v);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = rows(BR_D1 + 16 * wid, k);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) aW1[nt] += products(v, BR_X + 16 * nt);
    ab1 += sum(v);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = *reinterpret_cast<const f32x4 *>(lds.t + (BR_D3 + (r & 3)) * LDF + 4 * g + 16 * k);
      v[k] = r < NOUT ? v[k] : splat(0.0f);
    }
    aW3 += products(v, BR_H2 + 16 * wid);
    ab3 += sum(v);
    __syncthreads();  // the tiles are written again
  }
  // the block's partial
#pragma unroll
  for (int k = 16; k < 64; k <<= 1) {
    ab1 += __shfl_xor(ab1, k, 64);
    ab2 += __shfl_xor(ab2, k, 64);
    ab3 += __shfl_xor(ab3, k, 64);
  }
  float *out = partial + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = 16 * wid + 4 * g + i;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) out[OFF_W2 + m * NH + 16 * nt + r] = aW2[nt][i];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[OFF_W1 + m * NIN + 16 * nt + r] = aW1[nt][i];
    if (g == 0) out[OFF_W3 + i * NH + 16 * wid + r] = aW3[i];
  }
  if (g == 0) {
    out[OFF_B1 + 16 * wid + r] = ab1;
    out[OFF_B2 + 16 * wid + r] = ab2;
    if (wid == 0 && r < NOUT) out[OFF_B3 + r] = ab3;
  }
}

// --------------------------------------------------------------- BF16 bwd
// On BF16 MFMA 16x16x32 (FP32 accumulate), two waves to a SIMD.  An MFMA with
// its operands exchanged gives the
// transposed product from the same registers, out[sample 4g + i][neuron r] in
// place of out[neuron 4g + i][sample r]: each layer is computed in both, the
// first for the next layer, the second, four samples to a lane, for 8-byte
// stores to those tiles.
// 262,143 samples: 36 us.  A wave alone on a SIMD with every accumulator, 2-byte
// stores to its own tiles and loads at their use took 75 us: 6 of preparing
// weights, 7 us per 32 samples and 6 of adding the waves.
constexpr int LDB = kBwdSamples + 8;        // row stride of the sample tiles

struct BfBwdLds {
  union {
    float p[PO_SIZE];
    __bf16 t[BR_ROWS * LDB];
  };
  // fragments 2 mt + c of W2's transpose, 8 + 2 mt + c of W1's, 12 + mt of W1
  // (in registers all of them would not leave room for two waves on a SIMD)
  bf16x8 w[16][64];
  float b1[NH], b2[NH];
  float bias[kBwdWaves][9][16];
};

// Eight parameters, four each from p and q, as BF16.
__device__ __forceinline__ bf16x8 bf_halves(const float *p, const float *q) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(q);
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = (__bf16)a[j];
    v[4 + j] = (__bf16)b[j];
  }
  return v;
}

__device__ __forceinline__ bf16x8 pack_raw(const f32x4 z[4], int c) {
  bf16x8 b;
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = (__bf16)z[2 * c + j / 4][j % 4];
  return b;
}

struct BfIn {
  BfX x;
  float go;  // gradient of output g of sample r
};

template <bool kBone>
__device__ __forceinline__ void load_half(const uint32_t *feat, const float *go, const int16_t *bone, int64_t S,
                                          int64_t ld, int64_t s, int g, BfIn &in) {
  load_x<kBone>(feat, bone, S, ld, s, g, in.x);
  in.go = go[s < S ? s : S - 1];
}

// Values of four consecutive samples of a neuron, as BF16.
__device__ __forceinline__ void store_row4(__bf16 *t, int row, int col, const f32x4 &v) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 b;
#pragma unroll
  for (int i = 0; i < 4; ++i) b[i] = (__bf16)v[i];
  *reinterpret_cast<bf16x4 *>(t + row * LDB + col) = b;
}

__device__ __forceinline__ bf16x8 lds_row8(const __bf16 *t, int row, int col) {
  return *reinterpret_cast<const bf16x8 *>(t + row * LDB + col);
}

template <bool kBone>
__global__ void __launch_bounds__(kBwdBlock, 2) mlp_bwd_bf16(const float *__restrict__ gsig,
                                                            const float *__restrict__ grgb,
                                                            const __hip_bfloat16 *__restrict__ featb,
                                                            const int16_t *__restrict__ bone, int64_t S,
                                                            const int64_t *__restrict__ S_dev, int64_t ld,
                                                            const float *__restrict__ P, float *__restrict__ gfeat,
                                                            float *__restrict__ partial) {
  __shared__ __attribute__((aligned(16))) BfBwdLds lds;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const uint32_t *feat = reinterpret_cast<const uint32_t *>(featb);
  S = count_of(S, S_dev);
  const int64_t step = (int64_t)gridDim.x * kBwdSamples;
  const float *go = g == 0 ? gsig : grgb + (g - 1) * ld;
  int64_t s0 = (int64_t)blockIdx.x * kBwdSamples + 16 * wid;
  BfIn in = {};
  if (S > 0) load_half<kBone>(feat, go, bone, S, ld, s0 + r, g, in);
  stage_padded(P, lds.p);
  __syncthreads();
  const float *p = lds.p;
  bf16x8 w2[4][2], w3[2];
  float w3t[4], b1t[4], b2t[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float *q2 = p + PO_W2 + (16 * mt + r) * PW2 + 32 * c + 4 * g;
      w2[mt][c] = bf_halves(q2, q2 + 16);
    }
    b1t[mt] = p[PO_B1 + 16 * mt + r];
    b2t[mt] = p[PO_B2 + 16 * mt + r];
    w3t[mt] = (float)(__bf16)p[PO_W3 + g * PW3 + 16 * mt + r];
  }
  // rows 4k of the last layer's operand are W3's, the others zero, so that lane
  // (r, g) gets output g of sample r
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const float *q3 = p + PO_W3 + (r >> 2) * PW3 + 32 * c + 4 * g;
    const bf16x8 v = bf_halves(q3, q3 + 16), zero = {};
    w3[c] = (r & 3) == 0 ? v : zero;
  }
  const float b3 = p[PO_B3 + g];
  // the fragments in LDS, a quarter by each wave:
  // [16(2c + j/4) + 4g + j%4][16mt + r] of W2, W1; W1[16mt + r][8g + j]
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int q = kBwdWaves * k + wid, mt = (q & 7) >> 1, c = q & 1;
    const float *col = p + (k < 2 ? PO_W2 : PO_W1) + 16 * mt + r;
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)col[(16 * (2 * c + j / 4) + 4 * g + (j % 4)) * (k < 2 ? PW2 : PW1)];
    lds.w[q][lane] = v;
  }
  const float *q1 = p + PO_W1 + (16 * wid + r) * PW1 + 8 * g;
  lds.w[12 + wid][lane] = bf_halves(q1, q1 + 4);
  if (threadIdx.x < 2 * NH) (threadIdx.x < NH ? lds.b1 : lds.b2 - NH)[threadIdx.x] = p[PO_B1 + threadIdx.x];
  __syncthreads();  // the tiles take the parameters' place
  f32x4 aW1[2], aW2[4], aW3 = splat(0.0f);
  float ab1[4], ab2[4], ab3 = 0.0f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    ab1[a] = ab2[a] = 0.0f;
    aW2[a] = splat(0.0f);
    if (a < 2) aW1[a] = splat(0.0f);
  }
  const int col = 16 * wid + 4 * g;  // of the transposed products' samples
  for (int64_t b0 = (int64_t)blockIdx.x * kBwdSamples; b0 < S; b0 += step, s0 += step) {  // uniform in the block
    const int64_t s = s0 + r;
    const bool ok = s < S, use = ok && (!kBone || in.x.bone >= 0);
    bf16x8 X;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t v = ok ? in.x.x[j] : 0u;
      X[2 * j] = __builtin_bit_cast(__bf16, (uint16_t)(v & 0xffffu));
      X[2 * j + 1] = __builtin_bit_cast(__bf16, (uint16_t)(v >> 16));
      lds.t[(BR_X + 8 * g + 2 * j) * LDB + 16 * wid + r] = X[2 * j];
      lds.t[(BR_X + 8 * g + 2 * j + 1) * LDB + 16 * wid + r] = X[2 * j + 1];
    }
    const float go_s = in.go;
    // the next step's inputs (after the last: the last sample's again)
    load_half<kBone>(feat, go, bone, S, ld, s + step, g, in);
    // pre-activations and their transposes
    f32x4 z1[4], y1[4], z2[4], y2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 w1 = lds.w[12 + mt][lane];
      z1[mt] = mfma32(w1, X, *reinterpret_cast<const f32x4 *>(lds.b1 + 16 * mt + 4 * g));
      y1[mt] = mfma32(X, w1, splat(b1t[mt]));
    }
    const bf16x8 h1a = pack_act(z1, 0), h1b = pack_act(z1, 1);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      z2[mt] = mfma32(w2[mt][0], h1a, *reinterpret_cast<const f32x4 *>(lds.b2 + 16 * mt + 4 * g));
      z2[mt] = mfma32(w2[mt][1], h1b, z2[mt]);
      y2[mt] = mfma32(h1b, w2[mt][1], mfma32(h1a, w2[mt][0], splat(b2t[mt])));
    }
    f32x4 oa = {b3, 0.0f, 0.0f, 0.0f};
    oa = mfma32(w3[0], pack_act(z2, 0), oa);
    oa = mfma32(w3[1], pack_act(z2, 1), oa);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      f32x4 h1, h2;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h1[i] = relu(y1[mt][i]);
        h2[i] = relu(y2[mt][i]);
      }
      store_row4(lds.t, BR_H1 + 16 * mt + r, col, h1);
      store_row4(lds.t, BR_H2 + 16 * mt + r, col, h2);
    }
    // the gradient of output g of sample r
    const float o = oa[0], e = expf(g == 0 ? fminf(o, 80.0f) : -o), c = __builtin_amdgcn_rcpf(1.0f + e);
    float d3 = g == 0 ? (o < 80.0f ? go_s * e : 0.0f) : go_s * c * (1.0f - c);
    d3 = use ? d3 : 0.0f;
    ab3 += d3;
    lds.t[(BR_D3 + g) * LDB + 16 * wid + r] = (__bf16)d3;
    // the 4-wide head runs on FP32 MFMA with BF16-valued operands (the
    // forward's W3, the output delta as stored for the weight gradient)
    const float d3b = (float)(__bf16)d3;
    f32x4 d2[4], e2[4], d1[4], e1[4];  // deltas and their transposes
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      d2[mt] = mfma4(w3t[mt], d3b, splat(0.0f));
      e2[mt] = mfma4(d3b, w3t[mt], splat(0.0f));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d2[mt][i] = z2[mt][i] < 0.0f ? 0.0f : d2[mt][i];
        e2[mt][i] = y2[mt][i] < 0.0f ? 0.0f : e2[mt][i];
        ab2[mt] += e2[mt][i];
      }
      store_row4(lds.t, BR_D2 + 16 * mt + r, col, e2[mt]);
    }
    const bf16x8 d2a = pack_raw(d2, 0), d2b = pack_raw(d2, 1);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      const bf16x8 wa = lds.w[2 * mt][lane], wb = lds.w[2 * mt + 1][lane];
      d1[mt] = mfma32(wb, d2b, mfma32(wa, d2a, splat(0.0f)));
      e1[mt] = mfma32(d2b, wb, mfma32(d2a, wa, splat(0.0f)));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        d1[mt][i] = z1[mt][i] < 0.0f ? 0.0f : d1[mt][i];
        e1[mt][i] = y1[mt][i] < 0.0f ? 0.0f : e1[mt][i];
        ab1[mt] += e1[mt][i];
      }
      store_row4(lds.t, BR_D1 + 16 * mt + r, col, e1[mt]);
    }
    if (gfeat) {
      const bf16x8 d1a = pack_raw(d1, 0), d1b = pack_raw(d1, 1);
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const f32x4 acc = mfma32(lds.w[9 + 2 * mt][lane], d1b, mfma32(lds.w[8 + 2 * mt][lane], d1a, splat(0.0f)));
        if (ok) {
          float2 *gf = reinterpret_cast<float2 *>(gfeat);
          gf[(int64_t)(8 * mt + 2 * g) * ld + s] = make_float2(acc[0], acc[1]);
          gf[(int64_t)(8 * mt + 2 * g + 1) * ld + s] = make_float2(acc[2], acc[3]);
        }
      }
    }
    __syncthreads();
    // weight gradients of this wave's rows, K = the block's samples, summed from
    // zero so that the chains of roundings stay short
    auto rows = [&](int row, int k) { return lds_row8(lds.t, row + r, 32 * k + 8 * g); };
    const bf16x8 v1[2] = {rows(BR_D1 + 16 * wid, 0), rows(BR_D1 + 16 * wid, 1)};
    const bf16x8 v2[2] = {rows(BR_D2 + 16 * wid, 0), rows(BR_D2 + 16 * wid, 1)};
    bf16x8 v3[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bf16x8 zero = {}, v = lds_row8(lds.t, BR_D3 + (r & 3), 32 * k + 8 * g);
      v3[k] = r < NOUT ? v : zero;
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
      aW2[nt] += mfma32(v2[1], rows(BR_H1 + 16 * nt, 1), mfma32(v2[0], rows(BR_H1 + 16 * nt, 0), splat(0.0f)));
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
      aW1[nt] += mfma32(v1[1], rows(BR_X + 16 * nt, 1), mfma32(v1[0], rows(BR_X + 16 * nt, 0), splat(0.0f)));
    aW3 += mfma32(v3[1], rows(BR_H2 + 16 * wid, 1), mfma32(v3[0], rows(BR_H2 + 16 * wid, 0), splat(0.0f)));
    __syncthreads();  // the tiles are written again
  }
  // the block's partial: the weights as they are, the biases over the waves in
  // order (within a wave over the sample groups g, the last layer's over r)
#pragma unroll
  for (int k = 8; k > 0; k >>= 1) ab3 += __shfl_xor(ab3, k, 16);
#pragma unroll
  for (int k = 16; k < 64; k <<= 1)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      ab1[a] += __shfl_xor(ab1[a], k, 64);
      ab2[a] += __shfl_xor(ab2[a], k, 64);
    }
  if (g == 0)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      lds.bias[wid][a][r] = ab1[a];
      lds.bias[wid][4 + a][r] = ab2[a];
    }
  if (r == 0) lds.bias[wid][8][g] = ab3;
  float *out = partial + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = 16 * wid + 4 * g + i;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) out[OFF_W2 + m * NH + 16 * nt + r] = aW2[nt][i];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) out[OFF_W1 + m * NIN + 16 * nt + r] = aW1[nt][i];
    if (g == 0) out[OFF_W3 + i * NH + 16 * wid + r] = aW3[i];
  }
  __syncthreads();
  const int a = threadIdx.x / 16, q = threadIdx.x % 16;
  if (a < 8 || (a == 8 && q < NOUT)) {
    float v = lds.bias[0][a][q];
#pragma unroll
    for (int w = 1; w < kBwdWaves; ++w) v += lds.bias[w][a][q];
    out[a == 8 ? OFF_B3 + q : (a < 4 ? OFF_B1 : OFF_B2) + 16 * (a % 4) + q] = v;
  }
}

// Sum of the block partials per parameter: 64 parameters x 16 partial groups
// per workgroup; each thread sums its group in double with four independent
// accumulators, then the 16 groups are combined in a fixed order (the
// result does not depend on scheduling).
constexpr int kRedP = 64, kRedG = 16;
__global__ void __launch_bounds__(kRedP *kRedG) reduce_partials(const float *__restrict__ partial, int nblk,
                                                                float *__restrict__ out, int overwrite) {
  __shared__ double part[kRedG][kRedP];
  const int pl = threadIdx.x % kRedP, grp = threadIdx.x / kRedP;
  const int e = blockIdx.x * kRedP + pl;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  if (e < NPARAM) {
    int b = grp;
    for (; b + 3 * kRedG < nblk; b += 4 * kRedG) {
      a0 += (double)partial[(int64_t)b * NPARAM + e];
      a1 += (double)partial[(int64_t)(b + kRedG) * NPARAM + e];
      a2 += (double)partial[(int64_t)(b + 2 * kRedG) * NPARAM + e];
      a3 += (double)partial[(int64_t)(b + 3 * kRedG) * NPARAM + e];
    }
    for (; b < nblk; b += kRedG) a0 += (double)partial[(int64_t)b * NPARAM + e];
  }
  part[grp][pl] = (a0 + a1) + (a2 + a3);
  __syncthreads();
  if (grp == 0 && e < NPARAM) {
    double s = 0.0;
    for (int g = 0; g < kRedG; ++g) s += part[g][pl];
    out[e] = overwrite ? (float)s : out[e] + (float)s;
  }
}

// workgroups a CU holds by LDS: one for FP32, two for BF16
int bwd_blocks(int64_t S, int per_cu) {
  const int64_t b = ceil_div(S, (int64_t)kBwdSamples), most = 256 * per_cu;
  return b > most ? (int)most : (b < 1 ? 1 : (int)b);
}

// as many workgroups as stay resident, each wave looping over its tiles with
// the next tiles' loads in flight: two per CU for FP32 (180 registers a lane),
// four for BF16 (seven, which its 72 registers would allow, took 13.2 us for
// 262,143 samples against 12.0)
unsigned fwd_blocks(int64_t S, int per_cu) { return grid_for(ceil_div(S, 16) * 64, kMlpBlock, 256 * per_cu); }

}  // namespace

namespace {

// The one decoder shape the kernels implement (Eq. 1-2 with the widths of
// the Instant-NGP density/colour head): 32 -> 64 -> 64 -> 4.
int32_t widths_status(const int32_t *widths, int32_t n_layers) {
  if (!widths || n_layers < 1 || n_layers > 15) return IA355_ERR_INVALID_ARG;
  for (int l = 0; l <= n_layers; ++l)
    if (widths[l] <= 0) return IA355_ERR_INVALID_ARG;
  if (n_layers != 3 || widths[0] != NIN || widths[1] != NH || widths[2] != NH || widths[3] != NOUT)
    return IA355_ERR_UNSUPPORTED;
  return IA355_OK;
}

}  // namespace

extern "C" int32_t ia355_mlp_fwd(const void *feat, int32_t feat_dtype, const int16_t *bone, int64_t S,
                                 const int64_t *S_dev, int64_t ld, const float *params, const int32_t *widths,
                                 int32_t n_layers, int32_t dtype, float *sigma, float *rgb, ia355_stream_t stream) {
  const int32_t ws = widths_status(widths, n_layers);
  if (ws != IA355_OK) return ws;
  if (S < 0 || ld < S || !params || ((uintptr_t)params & 15)) return IA355_ERR_INVALID_ARG;
  if (S > 0 && (!feat || !sigma || !rgb)) return IA355_ERR_INVALID_ARG;
  if (dtype == IA355_F32 && feat_dtype != IA355_F32) return IA355_ERR_UNSUPPORTED;
  if (dtype == IA355_BF16 && feat_dtype != IA355_BF16) return IA355_ERR_UNSUPPORTED;
  if (dtype != IA355_F32 && dtype != IA355_BF16) return IA355_ERR_INVALID_ARG;
  if (S == 0) return IA355_OK;
  hipStream_t s = as_stream(stream);
  if (dtype == IA355_F32)
    (bone ? mlp_fwd_f32<true> : mlp_fwd_f32<false>)<<<fwd_blocks(S, 2), kMlpBlock, 0, s>>>(
        (const float *)feat, bone, S, S_dev, ld, params, sigma, rgb);
  else
    (bone ? mlp_fwd_bf16<true> : mlp_fwd_bf16<false>)<<<fwd_blocks(ceil_div(S, kBfTiles), 4), kMlpBlock, 0, s>>>(
        (const __hip_bfloat16 *)feat, bone, S, S_dev, ld, params, sigma, rgb);
  return launch_status();
}

extern "C" size_t ia355_mlp_bwd_workspace_size(int64_t S) {
  return align256(sizeof(float) * (size_t)NPARAM * bwd_blocks(S, 2));
}

extern "C" int32_t ia355_mlp_bwd(const float *grad_sigma, const float *grad_rgb, const void *feat, int32_t feat_dtype,
                                 const int16_t *bone, int64_t S, const int64_t *S_dev, int64_t ld,
                                 const float *params, const int32_t *widths, int32_t n_layers, int32_t dtype,
                                 float *grad_params, float *grad_feat, uint32_t flags, void *ws, size_t ws_bytes,
                                 ia355_stream_t stream) {
  const int32_t wst = widths_status(widths, n_layers);
  if (wst != IA355_OK) return wst;
  if (S < 0 || ld < S || !params || !grad_params || ((uintptr_t)params & 15)) return IA355_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)IA355_OVERWRITE) return IA355_ERR_INVALID_ARG;
  if (S > 0 && (!grad_sigma || !grad_rgb || !feat)) return IA355_ERR_INVALID_ARG;
  if (!((dtype == IA355_F32 && feat_dtype == IA355_F32) || (dtype == IA355_BF16 && feat_dtype == IA355_BF16)))
    return IA355_ERR_UNSUPPORTED;
  if (S == 0) return (flags & IA355_OVERWRITE) ? ia355_zero(grad_params, sizeof(float) * NPARAM, stream) : IA355_OK;
  if (!ws || ws_bytes < ia355_mlp_bwd_workspace_size(S)) return IA355_ERR_WORKSPACE;
  hipStream_t s = as_stream(stream);
  const int nb = bwd_blocks(S, dtype == IA355_F32 ? 1 : 2);
  if (dtype == IA355_F32) {
    auto fn = bone ? mlp_bwd_f32<true> : mlp_bwd_f32<false>;
    if (hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(F32BwdLds)) !=
        hipSuccess)
      return IA355_ERR_HIP;
    fn<<<nb, kBwdBlock, sizeof(F32BwdLds), s>>>(grad_sigma, grad_rgb, (const float *)feat, bone, S, S_dev, ld, params,
                                                grad_feat, (float *)ws);
  } else
    (bone ? mlp_bwd_bf16<true> : mlp_bwd_bf16<false>)<<<nb, kBwdBlock, 0, s>>>(
        grad_sigma, grad_rgb, (const __hip_bfloat16 *)feat, bone, S, S_dev, ld, params, grad_feat, (float *)ws);
  reduce_partials<<<(unsigned)ceil_div(NPARAM, kRedP), kRedP * kRedG, 0, s>>>((const float *)ws, nb, grad_params,
                                                                                     (flags & IA355_OVERWRITE) != 0);
  return launch_status();
}
