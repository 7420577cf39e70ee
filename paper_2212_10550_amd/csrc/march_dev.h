// Ray sampling with empty-space skipping (Sec. 3.2, Sec. 3.3), shared by the
// march kernels and the fused batch renderer so that both take the same
// keep/skip decisions and compute the same sample positions: every
// operation is an individually rounded IEEE single operation (internal).
#pragma once
#include <cmath>

#include "common.h"

namespace ia355 {
namespace mch {

struct Box {
  float lo[3], hi[3];
  float inv_ext[3];  // 1 / (hi - lo), used only when every extent is a power of two
};

struct RaySpan {
  float tn, tf, dt;
  bool hit;
};

__device__ __forceinline__ RaySpan ray_span(const float o[3], const float d[3], const Box &b, float dt_fixed,
                                            int n_per_ray) {
#pragma clang fp contract(off)
  float tmin = -INFINITY, tmax = INFINITY;
  RaySpan s{0.0f, 0.0f, 0.0f, false};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (d[a] != 0.0f) {
      const float ta = (b.lo[a] - o[a]) / d[a];
      const float tb = (b.hi[a] - o[a]) / d[a];
      const float t0 = ta < tb ? ta : tb;
      const float t1 = ta < tb ? tb : ta;
      if (t0 > tmin) tmin = t0;
      if (t1 < tmax) tmax = t1;
    } else if (o[a] < b.lo[a] || o[a] > b.hi[a]) {
      return s;
    }
  }
  const float tn = tmin > 0.0f ? tmin : 0.0f;
  if (!(tmax > tn)) return s;
  s.tn = tn;
  s.tf = tmax;
  s.dt = n_per_ray > 0 ? (tmax - tn) / (float)n_per_ray : dt_fixed;
  s.hit = true;
  return s;
}

// Ray parameter of step k: the midpoint of the k-th interval.
__device__ __forceinline__ float step_t(const RaySpan &s, int k) {
#pragma clang fp contract(off)
  return s.tn + ((float)k + 0.5f) * s.dt;
}

// Sample k of a ray: position and whether its cell is occupied.
// kPow2Ext: every box extent is a power of two, so dividing by it and
// multiplying by its (exact) reciprocal round the same real number once and
// give the same float; the multiply saves the division sequence.
template <bool kPow2Ext>
__device__ __forceinline__ bool sample_at(const float o[3], const float d[3], const RaySpan &s, int k, const Box &b,
                                          const uint32_t *bits, int G, float *t_out, float x[3]) {
#pragma clang fp contract(off)
  const float t = step_t(s, k);
  *t_out = t;
  int cell[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x[a] = o[a] + t * d[a];
    const float rel = kPow2Ext ? (x[a] - b.lo[a]) * b.inv_ext[a] : (x[a] - b.lo[a]) / (b.hi[a] - b.lo[a]);
    const float u = rel * (float)G;
    int c = (int)floorf(u);
    cell[a] = c < 0 ? 0 : (c > G - 1 ? G - 1 : c);
  }
  if (!bits) return true;
  const uint32_t word = occ_word(cell[0], cell[1], cell[2], G);
  return (bits[word] >> occ_bit(cell[0], cell[1])) & 1u;
}

// How a box maps to its grid: kGeneral divides by the extents; kPow2 (every
// extent a power of two) multiplies by inv_ext G, which is exact and rounds
// the same product once; kPow2AtZero is that with the low corner at zero,
// where x - lo is x.
enum BoxKind { kGeneral, kPow2, kPow2AtZero };

// Cell of the sample at ray parameter t, as sample_at finds it.  The clamp to
// [0, G - 1] comes before the truncation, which then equals floor and clamp
// (v_med3_f32; a NaN ends in some cell, as it does there).
template <BoxKind kBox>
__device__ __forceinline__ void sample_cell(const float o[3], const float d[3], float t, const Box &b, int G,
                                            uint32_t cell[3]) {
#pragma clang fp contract(off)
  const float top = (float)(G - 1);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float x = o[a] + t * d[a];
    const float rel = kBox == kPow2AtZero ? x : x - b.lo[a];
    const float u = kBox == kGeneral ? rel / (b.hi[a] - b.lo[a]) * (float)G : rel * (b.inv_ext[a] * (float)G);
    cell[a] = (uint32_t)__builtin_amdgcn_fmed3f(u, 0.0f, top);
  }
}

// Byte of the packed grid that holds cell (x, y, z) (its bit is x mod 8);
// sy, sz: bytes of a row and of a layer of bricks (< 2^24 for G <= 2048).
__device__ __forceinline__ uint32_t occ_byte(uint32_t x, uint32_t y, uint32_t z, uint32_t sy, uint32_t sz) {
  const uint32_t row = __umul24(y >> 3, sy) + ((x >> 3) << 7);
  return __umul24(z >> 4, sz) + row + (((z & 15u) << 3) | (y & 7u));
}

// Position of the q-th (from 0) set bit of m; q < the number of set bits.
__device__ __forceinline__ int select_bit64(uint64_t m, int q) {
  const uint32_t lo = (uint32_t)m;
  const int c0 = __popc(lo);
  uint32_t v = q < c0 ? lo : (uint32_t)(m >> 32);
  int pos = q < c0 ? 0 : 32;
  q = q < c0 ? q : q - c0;
#pragma unroll
  for (int w = 16; w >= 1; w >>= 1) {
    const int c = __popc(v & ((1u << w) - 1u));
    const bool up = q >= c;
    q = up ? q - c : q;
    v = up ? v >> w : v;
    pos = up ? pos + w : pos;
  }
  return pos;
}

__device__ __forceinline__ void load_ray(const float *ro, const float *rd, int64_t r, float o[3], float d[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    o[a] = ro[3 * r + a];
    d[a] = rd[3 * r + a];
  }
}

// Position and ray parameter of step k (the expressions of sample_at).
__device__ __forceinline__ void sample_pos(const float o[3], const float d[3], float tn, float dt, int k, float *t_out,
                                           float x[3]) {
#pragma clang fp contract(off)
  const float t = tn + ((float)k + 0.5f) * dt;
  *t_out = t;
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = o[a] + t * d[a];
}

// Host side: the occupancy box, and whether every extent is a power of two
// (then sample_at may multiply by the exact reciprocal).  False for an empty
// or inverted box.
inline bool make_box(const float *aabb, Box *box, bool *pow2) {
  if (!aabb) return false;
  for (int a = 0; a < 3; ++a) {
    box->lo[a] = aabb[a];
    box->hi[a] = aabb[3 + a];
    if (!(box->hi[a] > box->lo[a])) return false;
  }
  bool p2 = true;
  for (int a = 0; a < 3; ++a) {
    const float ext = box->hi[a] - box->lo[a];
    int e;
    p2 = p2 && std::isfinite(ext) && std::frexp(ext, &e) == 0.5f && e > -100 && e < 100;
    box->inv_ext[a] = p2 ? 1.0f / ext : 0.0f;
  }
  *pow2 = p2;
  return true;
}

}  // namespace mch
}  // namespace ia355
