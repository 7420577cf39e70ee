// Learned root initialiser for the canonical-correspondence search (an
// addition to the root finding of Sec. 3.1, not in the paper): a small MLP maps
// (posed point x', pose) to per-bone logits and a canonical offset; the
// start point handed to Broyden is x0 = B_k^{-1} x' + offset, k = argmax.
//
// Layer 1 takes (x', pose); the pose part W1[:, 3:] pose + b1 is the same
// for every sample of a pose, so each workgroup folds it into a per-neuron
// constant once and layer 1 costs 3 FMAs per neuron.  Layers 2 and 3 run on
// MFMA exactly like the decoder MLP (one wave per 16-sample tile, the
// hidden activations chained in registers through the K ordering), in FP32
// (16x16x4) or BF16 (16x16x32, FP32 accumulate).  The argmax over the bone
// logits is a cross-lane reduction.
#include "common.h"
#include "geometry.h"
#include "rootinit_dev.h"

using namespace ia355;

namespace {

constexpr int kBlock = 256;
using rid::H;
using rid::kMaxOut;

// FP32: the whole parameter block is staged in LDS (61.5 KB, coalesced 16-byte
// loads; the pose fold walks W1 row by row, the MFMA fragments gather single
// values) and the fragments held in registers.
__global__ void __launch_bounds__(kBlock, 1) rootinit_f32(const float *__restrict__ xp_soa, int64_t S,
                                                          const int64_t *__restrict__ S_dev, int64_t ld,
                                                          const float *__restrict__ pose, const float *__restrict__ P,
                                                          const float *__restrict__ B, int nb,
                                                          int16_t *__restrict__ bone_out, float *__restrict__ x0_soa) {
  const rid::Layout l = rid::layout(nb);
  // a block without a tile returns before any work (uniform, ahead of the
  // barriers): with a device-side count the grid is sized for the capacity
  S = count_of(S, S_dev);
  if ((int64_t)blockIdx.x * (kBlock / 64) >= ceil_div(S, 16)) return;
  __shared__ float c1[H];        // W1[:, 3:] pose + b1
  __shared__ float w1x[H * 3];   // W1[:, :3]
  __shared__ float sBinv[64 * 12];
  __shared__ int sBok[64];
  extern __shared__ __attribute__((aligned(16))) float sP[];
  static_assert(kBlock == 4 * H, "four threads per hidden neuron");
  rid::stage_copy(P, l.total, sP);
  __syncthreads();
  rid::fold_pose(sP, l, pose, nb, c1);
  for (int e = threadIdx.x; e < H * 3; e += kBlock) w1x[e] = sP[l.offW1 + (e / 3) * l.nin + (e % 3)];
  stage_bone_inverses(B, nb, sBinv, sBok);
  __syncthreads();

  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  rid::Frag f;
  rid::load_frag(sP, l, r, g, f);
  const int64_t ntile = ceil_div(S, 16);
  const int64_t wstride = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t tile = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); tile < ntile; tile += wstride) {
    const int64_t s = tile * 16 + r;
    const bool ok = s < S;
    float x[3] = {0.0f, 0.0f, 0.0f};
    if (ok) {
      x[0] = xp_soa[s];
      x[1] = xp_soa[ld + s];
      x[2] = xp_soa[2 * ld + s];
    }
    int bi;
    float off[3];
    rid::tile_f32(x, c1, w1x, f, nb, g, &bi, off);
    if (g == 0 && ok) {
      const int k = bi < nb ? bi : 0;
      bone_out[s] = (int16_t)k;
      float x0[3];
      rid::start_point(sBinv + 12 * k, x, off, x0);
#pragma unroll
      for (int a = 0; a < 3; ++a) x0_soa[a * ld + s] = x0[a];
    }
  }
}

// BF16: the parameters are read from global memory once per block (the pose
// fold, layer 1's x weights, the layer 2-3 fragments into a 12 KB LDS store
// read as the MFMAs need them).  A wave takes 64 samples a step, or 32 in a
// call (or a device count) too small to give every SIMD a wave of 64 and then
// some: one per lane for the points, the start points and the stores, and in
// pairs of 16-sample tiles for the layers, so that each LDS read of weights
// serves two.
// 875,600 samples: 34 us.  A tile at a time (34 16-byte LDS reads each,
// branches in the argmax, sixteen lanes at the start points, staging that
// waited for every load) took 43 us.
// The line between the steps: 64 samples 7.8 -> 6.7 us with 32 a step, 16,384
// 8.3 -> 7.2, 32,768 8.4 -> 7.3, a count of 5000 under a capacity of 200,000
// 8.3 -> 7.2; 65,536 8.7 either way.
constexpr int kPair = 2;
constexpr int64_t kOnePairSamples = 32768;

__global__ void __launch_bounds__(kBlock, 4) rootinit_bf16(const float *__restrict__ xp_soa, int64_t S,
                                                           const int64_t *__restrict__ S_dev, int64_t ld,
                                                           const float *__restrict__ pose, const float *__restrict__ P,
                                                           const float *__restrict__ B, int nb,
                                                           int16_t *__restrict__ bone_out, float *__restrict__ x0_soa) {
  const rid::Layout l = rid::layout(nb);
  S = count_of(S, S_dev);
  const int pairs = S <= kOnePairSamples ? 1 : 2, kStep = 16 * kPair * pairs;
  const int64_t nstep = ceil_div(S, (int64_t)kStep), wstride = (int64_t)gridDim.x * (kBlock / 64);
  if ((int64_t)blockIdx.x * (kBlock / 64) >= nstep) return;  // as above
  __shared__ __attribute__((aligned(16))) float c1[H];       // W1[:, 3:] pose + b1
  __shared__ __attribute__((aligned(16))) float w1x[H * 3];  // W1[:, :3]
  __shared__ float sBinv[64 * 12];
  __shared__ int sBok[64];
  __shared__ __attribute__((aligned(16))) bf16x8 sRw[12][kWave];
  __shared__ __attribute__((aligned(16))) float sRb2[H], sRb3[kMaxOut];
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  int64_t st = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  float xn[3];  // the next step's point, from a valid index in any case
  auto load = [&](int64_t s) {
    s = s < S ? s : S - 1;
#pragma unroll
    for (int a = 0; a < 3; ++a) xn[a] = xp_soa[a * ld + s];
  };
  load(st * kStep + (lane & kStep - 1));
  rid::stage_frag_lds(P, l, sRw, sRb2, sRb3);
  rid::fold_pose(P, l, pose, nb, c1);
  for (int e = threadIdx.x; e < H * 3; e += kBlock) w1x[e] = P[l.offW1 + (e / 3) * l.nin + (e % 3)];
  stage_bone_inverses(B, nb, sBinv, sBok);
  __syncthreads();

  const rid::LdsFragW w{sRw, sRb2, sRb3, lane, g};
  for (; st < nstep; st += wstride) {
    const int64_t s = st * kStep + (lane & kStep - 1);
    float x[3], off[3] = {0.0f, 0.0f, 0.0f};
    int bi = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) x[a] = xn[a];
    load(s + wstride * kStep);
    for (int p = 0; p < pairs; ++p) {
      // the weights' reads stay in the loop (hoisted, they would hold every
      // fragment in registers)
      asm volatile("" ::: "memory");
      float xs[kPair][3];
#pragma unroll
      for (int u = 0; u < kPair; ++u)
#pragma unroll
        for (int a = 0; a < 3; ++a) xs[u][a] = __shfl(x[a], 16 * (kPair * p + u) + r, 64);
      bf16x8 h[kPair][2];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float cw[4], wx[12];
        *reinterpret_cast<f32x4 *>(cw) = *reinterpret_cast<const f32x4 *>(c1 + 16 * t + 4 * g);
#pragma unroll
        for (int q = 0; q < 3; ++q)
          *reinterpret_cast<f32x4 *>(wx + 4 * q) = *reinterpret_cast<const f32x4 *>(w1x + 3 * (16 * t + 4 * g) + 4 * q);
#pragma unroll
        for (int u = 0; u < kPair; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            h[u][t / 2][4 * (t % 2) + i] = (__bf16)rid::neuron1(xs[u], cw[i], wx + 3 * i);
      }
      f32x4 z[kPair][4], o[kPair][2];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const bf16x8 a0 = w.w2(mt, 0), a1 = w.w2(mt, 1);
        const f32x4 b = w.b2(mt);
#pragma unroll
        for (int u = 0; u < kPair; ++u) {
          z[u][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, h[u][0], b, 0, 0, 0);
          z[u][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, h[u][1], z[u][mt], 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < kPair; ++u)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          h[u][0][j] = (__bf16)rid::relu(z[u][j / 4][j % 4]);
          h[u][1][j] = (__bf16)rid::relu(z[u][2 + j / 4][j % 4]);
        }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const bf16x8 a0 = w.w3(mt, 0), a1 = w.w3(mt, 1);
        const f32x4 b = w.b3(mt);
#pragma unroll
        for (int u = 0; u < kPair; ++u) {
          o[u][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, h[u][0], b, 0, 0, 0);
          o[u][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, h[u][1], o[u][mt], 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < kPair; ++u) {
        int bt;
        float ot[3];
        rid::pick(o[u], nb, g, &bt, ot);
        const bool mine = g == kPair * p + u;  // lane r + 16 g keeps tile g's sample r
        bi = mine ? bt : bi;
#pragma unroll
        for (int a = 0; a < 3; ++a) off[a] = mine ? ot[a] : off[a];
      }
    }
    const int k = bi < nb ? bi : 0;
    float x0[3];
    rid::start_point(sBinv + 12 * k, x, off, x0);
    if (s < S && lane < kStep) {
      bone_out[s] = (int16_t)k;
#pragma unroll
      for (int a = 0; a < 3; ++a) x0_soa[a * ld + s] = x0[a];
    }
  }
}

}  // namespace

extern "C" int32_t ia355_rootinit_fwd(const float *xp, int64_t S, const int64_t *S_dev, int64_t ld, const float *pose,
                                      const float *params,
                                      int32_t hidden, const float *B, int32_t nb, int32_t dtype, int16_t *init_bone,
                                      float *x0, ia355_stream_t stream) {
  if (S < 0 || ld < S || nb <= 0 || !pose || !params || !B) return IA355_ERR_INVALID_ARG;
  if (hidden != H || nb + 3 > kMaxOut) return IA355_ERR_UNSUPPORTED;
  if (dtype != IA355_F32 && dtype != IA355_BF16) return IA355_ERR_INVALID_ARG;
  if (S > 0 && (!xp || !init_bone || !x0)) return IA355_ERR_INVALID_ARG;
  if (S == 0) return IA355_OK;
  // FP32: at most two blocks per CU (the parameters take 61.5 KB of LDS
  // each); BF16: four; each wave loops over its tiles
  const size_t lds = sizeof(float) * (size_t)(H * (3 + 6 * nb) + H + H * H + H + (nb + 3) * H + (nb + 3));
  if (lds > 96 * 1024) return IA355_ERR_UNSUPPORTED;
  hipStream_t s = as_stream(stream);
  if (dtype == IA355_F32)
    rootinit_f32<<<grid_for(ceil_div(S, 16) * 64, kBlock, 256 * 2), kBlock, lds, s>>>(
        xp, S, S_dev, ld, pose, params, B, nb, init_bone, x0);
  else
    rootinit_bf16<<<grid_for(S <= kOnePairSamples ? 2 * S : S, kBlock, 256 * 4), kBlock, 0, s>>>(
        xp, S, S_dev, ld, pose, params, B, nb, init_bone, x0);
  return launch_status();
}
