// Ray marching with empty-space skipping (Sec. 3.2 ray sampling, Sec. 3.3
// occupancy-grid skipping), as a stream compaction in four kernels:
//   count  -- which midpoint samples of each ray lie in occupied cells (a
//             keep mask, 64 steps a word), the ray's count and the block's
//             total: one wave per ray and one lane per sample for few rays,
//             one lane per ray for many;
//   chunk  -- each block scans 8192 block totals (exclusive, in place; one
//             block of 1024 or 4096 where that is all) and writes its chunk
//             total;
//   top    -- one block scans the chunk totals and writes the sample count
//             (skipped when there is one chunk: the chunk kernel writes it);
//   fill   -- from the keep masks and the ray's entry distance: only kept
//             samples' positions are recomputed (the same expression, so the
//             same floats), no cell lookups.  Few rays: one wave per ray, a
//             kept sample's slot is the ray's offset plus the popcount of kept
//             lanes below it.  Many rays: a wave takes the samples of its 64
//             rays, which are consecutive in the output, 64 at a time, a lane
//             finding its ray and step from its slot.  A ray's samples are
//             written in t order by consecutive lanes either way
//             (structure-of-arrays, coalesced).
// The occupancy bits are stored in bricks of 8 x 8 x 16 cells, one 128-byte
// cache line each, so the consecutive samples of a ray (one wave) touch a
// few lines rather than one line per sample.
// Every position and keep/skip decision is computed with individually
// rounded IEEE single operations (contraction is switched off: the
// compiler would otherwise fuse o + t d into one FMA), so the sample set is
// exactly reproducible.
#include <cmath>

#include "common.h"
#include "march_dev.h"

using namespace ia355;
using namespace ia355::mch;

namespace {

// Two mappings, by the ray count.  Few rays (a training step's thousands): one
// ray per wave, four waves per workgroup, lane l takes steps l, l + 64, ...,
// so that there are enough waves.  Many: one ray per lane, 256 per workgroup.
// An image's neighbouring rays walk neighbouring cells, so the 64 loads of a
// step touch a few lines, no lane is spent on steps past the box (a 128-step
// ray crosses a unit box in 74 steps at most), the ray clip with its six
// divisions is done once per ray instead of once per lane, and the fill's waves
// are full although a ray keeps only 3 samples on average.
// 1080^2 rays, 128^3 grid, 10 % occupied: count 358 -> 56 us, fill 194 -> 29
// us against four rays per wave.  The line lies where the two cross: a lane's
// chain of steps takes as long for one ray as for thousands, a wave per ray as
// much as there are rays.  Whole march, us, wave / lane per ray, up to 128
// steps: 16,384 rays 17-19 / 16-23, 20,480 21-23 / 16-23, 32,767 29-32 / 19-24
// (an image with and without a grid, a general box, random directions); of 600
// steps: 32,767 rays 54 / 80, 65,536 95 / 83.
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWavesPerBlock * kWave;
constexpr int64_t kManyRays = 20480, kAnyManyRays = 65536;
constexpr int kManySteps = 1 << 22;  // step indices plus a half are exact in single

// likely: the steps of a ray of unit direction along the box's diagonal
inline bool many_rays(int64_t R, int max_steps, const float *aabb, float dt, int n_per_ray) {
  const double ex = (double)aabb[3] - aabb[0], ey = (double)aabb[4] - aabb[1], ez = (double)aabb[5] - aabb[2];
  const double likely = n_per_ray > 0 ? (double)n_per_ray : sqrt(ex * ex + ey * ey + ez * ez) / (double)dt;
  const double steps = likely < (double)max_steps ? likely : (double)max_steps;
  const double line = (double)kManyRays + (steps > 128.0 ? 32.0 * (steps - 128.0) : 0.0);
  return max_steps <= kManySteps && ((double)R >= line || R >= kAnyManyRays);
}
// Waves that share 64 rays in the fill of many rays: enough for 16,384 in all
// (a wave's slots come one after the other), at most 16.
inline unsigned fill_parts(int64_t R) {
  const int64_t n = ((int64_t)1 << 20) / R;
  return (unsigned)(n < 1 ? 1 : n > 16 ? 16 : n);
}

template <bool kPow2Ext>
__global__ void __launch_bounds__(kBlock) march_count(const float *ro, const float *rd, int64_t R,
                                                      const uint32_t *bits, int G, Box box, float dt_fixed,
                                                      int n_per_ray, int max_steps, int64_t *ray_off,
                                                      int32_t *ray_cnt, float *ray_dt, int64_t *block_sum,
                                                      uint64_t *masks, int nw, float *ray_tn) {
  __shared__ int cnts[kWavesPerBlock];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int64_t r0 = (int64_t)blockIdx.x * kWavesPerBlock + wid;
  float o[3], d[3];
  load_ray(ro, rd, r0 < R ? r0 : R - 1, o, d);  // a tail wave repeats the last ray, writes nothing for it
  const RaySpan s = ray_span(o, d, box, dt_fixed, n_per_ray);
  int cnt = 0;
  for (int w0 = 0; w0 < nw; w0 += 2) {
    bool keep[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = (w0 + h) * kWave + lane;
      float t = 0.0f, x[3];
      keep[h] = false;
      // a step past t_far is not kept, so its cell is not looked up
      if (s.hit && k < max_steps && step_t(s, k) < s.tf)
        keep[h] = sample_at<kPow2Ext>(o, d, s, k, box, bits, G, &t, x) && t < s.tf;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint64_t m = __ballot(keep[h]);
      cnt += __popcll(m);
      if (lane == 0 && r0 < R && w0 + h < nw) masks[r0 * nw + w0 + h] = m;
    }
  }
  if (lane == 0) {
    if (r0 < R) {
      ray_cnt[r0] = cnt;
      ray_dt[r0] = s.dt;
      ray_tn[r0] = s.tn;
    }
    cnts[wid] = r0 < R ? cnt : 0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t acc = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      const int64_t ri = (int64_t)blockIdx.x * kWavesPerBlock + i;
      if (ri < R) ray_off[ri] = acc;
      acc += cnts[i];
    }
    block_sum[blockIdx.x] = acc;
  }
}

// One lane per ray.  kStepsAhead steps' occupancy bytes (8 cells along x) are
// loaded together.  Bound by instruction issue: about 40 per step and wave.
constexpr int kStepsAhead = 8;
// From this number of rays left on, a wave takes them one after the other, a
// step per lane: 64 steps cost it some 60 instructions a ray, against 2500 for
// all (65,536 rays of differing lengths, up to 1024 steps: 98 us -> 26).
constexpr int kFewLive = 24;

template <BoxKind kBox, bool kSkip>
__global__ void __launch_bounds__(kBlock) march_count_many(const float *__restrict__ ro, const float *__restrict__ rd,
                                                           int64_t R, const uint8_t *__restrict__ bits, int G, Box box,
                                                           float dt_fixed, int n_per_ray, int max_steps,
                                                           int64_t *__restrict__ ray_off, int32_t *__restrict__ ray_cnt,
                                                           float *__restrict__ ray_dt, int64_t *__restrict__ block_sum,
                                                           uint64_t *__restrict__ masks, int nw,
                                                           float *__restrict__ ray_tn) {
#pragma clang fp contract(off)
  __shared__ int wsum[kWavesPerBlock];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  float o[3], d[3];
  load_ray(ro, rd, r < R ? r : R - 1, o, d);
  const RaySpan s = ray_span(o, d, box, dt_fixed, n_per_ray);
  const float tf = s.hit && r < R ? s.tf : -INFINITY;
  const uint32_t nb = (uint32_t)(G + 7) >> 3, sy = nb << 7, sz = nb * sy;
  int cnt = 0;
  // t never falls along a ray, so once a step is past t_far for every lane
  // all later ones are
  bool live = true;
  for (int w = 0; w < nw; ++w) {
    uint32_t m[2] = {0u, 0u};
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 32 / kStepsAhead; ++c) {
        const int k0 = w * kWave + h * 32 + c * kStepsAhead;
        live = live && k0 < max_steps && __any(step_t(s, k0) < tf);
        if (!live) continue;
        // step_t of k0 + j: k0 + 1/2 + j is exact (max_steps <= kManySteps)
        const float kf = (float)k0 + 0.5f;
        uint32_t v[kStepsAhead], cx[kStepsAhead];
        bool in[kStepsAhead];
#pragma unroll
        for (int j = 0; j < kStepsAhead; ++j) {
          uint32_t cell[3];
          const float t = s.tn + (kf + (float)j) * s.dt;
          in[j] = k0 + j < max_steps && t < tf;
          sample_cell<kBox>(o, d, t, box, G, cell);
          cx[j] = cell[0];
          // read past the span too: any position is clamped to a cell
          v[j] = kSkip ? bits[occ_byte(cell[0], cell[1], cell[2], sy, sz)] : 0xffu;
        }
#pragma unroll
        for (int j = 0; j < kStepsAhead; ++j) {
          const uint32_t bit = in[j] ? (v[j] >> (cx[j] & 7u)) & 1u : 0u;
          m[h] |= bit << (c * kStepsAhead + j);
        }
      }
    cnt += __popc(m[0]) + __popc(m[1]);
    if (r < R) masks[r * nw + w] = (uint64_t)m[0] | (uint64_t)m[1] << 32;
    // the rays that go on; the fill reads no word past a ray's last kept step
    uint64_t on = w + 1 < nw ? __ballot(step_t(s, (w + 1) * kWave) < tf) : 0ull;
    if (on == 0ull) break;
    // few rays go on, and one of them for more groups of steps than there are
    // such rays: one after the other, a step per lane
    const int few = __popcll(on);
    if (few > kFewLive || !__any(step_t(s, (w + 1) * kWave + kStepsAhead * few) < tf)) continue;
    for (; on != 0ull; on &= on - 1ull) {
      const int u = __builtin_ctzll(on);
      auto of = [&](float v) { return __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(v), u)); };
      const float uo[3] = {of(o[0]), of(o[1]), of(o[2])}, ud[3] = {of(d[0]), of(d[1]), of(d[2])};
      const float un = of(s.tn), uf = of(tf), udt = of(s.dt);
      int kept = 0;
      for (int q = w + 1; q < nw; ++q) {
        const int k = q * kWave + lane;
        const float t = un + ((float)k + 0.5f) * udt;
        uint32_t cell[3];
        sample_cell<kBox>(uo, ud, t, box, G, cell);
        const uint32_t v = kSkip ? bits[occ_byte(cell[0], cell[1], cell[2], sy, sz)] : 0xffu;
        const uint64_t keep = __ballot(k < max_steps && t < uf && ((v >> (cell[0] & 7u)) & 1u));
        if (lane == u) masks[r * nw + q] = keep;
        kept += __popcll(keep);
        if (__ballot(t < uf) != ~0ull) break;
      }
      cnt += lane == u ? kept : 0;
    }
    break;
  }
  const int incl = wave_incl_scan(cnt);
  if (lane == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kWavesPerBlock; ++i) {
    base += i < wid ? wsum[i] : 0;
    all += wsum[i];
  }
  if (r < R) {
    ray_off[r] = base + incl - cnt;
    ray_cnt[r] = cnt;
    ray_dt[r] = s.dt;
    ray_tn[r] = s.tn;
  }
  if (threadIdx.x == 0) block_sum[blockIdx.x] = all;
}

// Exclusive scan in one block of 1024 threads: thread t holds `v`; returns
// the sum of the values of threads below it, and the block total in *total.
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t *wsum, int64_t *total) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  int64_t incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  if (lane == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  int64_t base = 0, all = 0;
  for (int w = 0; w < 1024 / kWave; ++w) {
    base += w < wid ? wsum[w] : 0;
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return base + incl - v;
}

// Chunk c of the per-block totals, kPer per thread: exclusive scan in place
// (offsets within the chunk) and the chunk's total.  kScanPer a thread where
// there are several chunks; a single one takes as few as hold it (a thread's
// totals are loaded and stored 8 bytes at a time, kPer apart).
constexpr int kScanPer = 8;  // one chunk holds 2 M rays at 256 a block
constexpr int64_t kScanChunk = 1024 * kScanPer;

template <int kPer>
__global__ void __launch_bounds__(1024) march_scan_chunk(int64_t *block_sum, int64_t nblk, int64_t *chunk_sum,
                                                         int64_t *ray_off, int64_t R, int64_t *n_samples) {
  __shared__ int64_t wsum[1024 / kWave];
  const int64_t i0 = (int64_t)blockIdx.x * 1024 * kPer + (int64_t)threadIdx.x * kPer;
  int64_t v[kPer], run = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    v[j] = i0 + j < nblk ? block_sum[i0 + j] : 0;
    run += v[j];
  }
  int64_t total;
  int64_t off = block_exclusive_scan(run, wsum, &total);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (i0 + j < nblk) block_sum[i0 + j] = off;
    off += v[j];
  }
  if (threadIdx.x == 0) {
    chunk_sum[blockIdx.x] = total;
    if (gridDim.x == 1) {  // a single chunk: its total is the sample count
      chunk_sum[0] = 0;
      n_samples[0] = total;
      ray_off[R] = total;
    }
  }
}

// Exclusive scan of the chunk totals (in place) in one block; the grand
// total goes to n_samples and ray_off[R].
__global__ void __launch_bounds__(1024) march_scan_top(int64_t *chunk_sum, int64_t nchunk, int64_t *ray_off,
                                                       int64_t R, int64_t *n_samples) {
  __shared__ int64_t wsum[1024 / kWave];
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < nchunk; c0 += 1024) {
    const int64_t i = c0 + threadIdx.x;
    const int64_t v = i < nchunk ? chunk_sum[i] : 0;
    int64_t total;
    const int64_t off = block_exclusive_scan(v, wsum, &total);
    if (i < nchunk) chunk_sum[i] = carry + off;
    carry += total;
  }
  if (threadIdx.x == 0) {
    n_samples[0] = carry;
    ray_off[R] = carry;
  }
}

__global__ void __launch_bounds__(kBlock) march_fill(const float *__restrict__ ro, const float *__restrict__ rd,
                                                     int64_t R, const uint64_t *__restrict__ masks, int nw,
                                                     const float *__restrict__ ray_tn, const int64_t *block_off,
                                                     const int64_t *chunk_off, int64_t *ray_off,
                                                     const float *__restrict__ ray_dt, float *xs, float *ts,
                                                     int32_t *ray_id, int64_t cap) {
  // the wave index is uniform: a ray's inputs and masks go through the
  // scalar cache
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int64_t r = (int64_t)blockIdx.x * kWavesPerBlock + wid;
  if (r >= R) return;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
  float o[3], d[3];
  load_ray(ro, rd, r, o, d);
  const float tn = ray_tn[r], dt = ray_dt[r];
  int64_t at0 = ray_off[r] + block_off[blockIdx.x] + chunk_off[blockIdx.x / kScanChunk];
  __builtin_amdgcn_wave_barrier();
  if (lane == 0) ray_off[r] = at0;
  const uint64_t *mr = masks + r * nw;
  for (int w = 0; w < nw; ++w) {
    const uint64_t m = mr[w];
    if (m == 0ull) continue;
    if ((m >> lane) & 1ull) {
      const int64_t at = at0 + __popcll(m & below);
      if (at < cap) {
        float t, x[3];
        sample_pos(o, d, tn, dt, w * kWave + lane, &t, x);
        xs[at] = x[0];
        xs[cap + at] = x[1];
        xs[2 * cap + at] = x[2];
        ts[at] = t;
        ray_id[at] = (int32_t)r;
      }
    }
    at0 += __popcll(m);
  }
}

// Many rays: gridDim.y waves write the samples of 64 rays, 64 slots at a time
// each.  The rays' first slots and inputs are in LDS; a lane finds its ray by
// binary search and its step as the q-th set bit of the ray's masks (global
// memory, read in the cache line of the neighbouring lanes' rays).
__global__ void __launch_bounds__(kBlock) march_fill_many(const float *__restrict__ ro, const float *__restrict__ rd,
                                                          int64_t R, const uint64_t *__restrict__ masks, int nw,
                                                          const float *__restrict__ ray_tn,
                                                          const int64_t *__restrict__ block_off,
                                                          const int64_t *__restrict__ chunk_off,
                                                          int64_t *__restrict__ ray_off,
                                                          const int32_t *__restrict__ ray_cnt,
                                                          const float *__restrict__ ray_dt, float *__restrict__ xs,
                                                          float *__restrict__ ts, int32_t *__restrict__ ray_id,
                                                          int64_t cap) {
  __shared__ float in[kWavesPerBlock][8][kWave];        // o, d, tn, dt of the wave's rays
  __shared__ int first[kWavesPerBlock][kWave];          // first slot of each ray, from the wave's first
  const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int64_t r0 = (int64_t)blockIdx.x * kBlock + wid * kWave;
  if (r0 >= R) return;  // no barrier below: a wave works alone
  const int64_t r = r0 + lane;
  const int cnt = r < R ? ray_cnt[r] : 0;
  int above = 0;  // of the block's rays before the wave's (the offsets in ray_off change meanwhile)
#pragma unroll
  for (int i = 1; i < kWavesPerBlock; ++i) above += i <= wid ? ray_cnt[r - i * kWave < R ? r - i * kWave : R - 1] : 0;
  const int incl = wave_incl_scan(cnt);
  const int n = __builtin_amdgcn_readlane(incl, kWave - 1);
  const int64_t at0 = block_off[blockIdx.x] + chunk_off[blockIdx.x / kScanChunk] +
                      __builtin_amdgcn_readlane(wave_incl_scan(above), kWave - 1);
  if (r < R && blockIdx.y == 0) ray_off[r] = at0 + incl - cnt;
  const int j0 = (int)blockIdx.y * kWave, step = (int)gridDim.y * kWave;
  if (j0 >= n) return;
  {
    float o[3], d[3];
    const int64_t q = r < R ? r : R - 1;
    load_ray(ro, rd, q, o, d);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      in[wid][a][lane] = o[a];
      in[wid][3 + a][lane] = d[a];
    }
    in[wid][6][lane] = ray_tn[q];
    in[wid][7][lane] = ray_dt[q];
    first[wid][lane] = incl - cnt;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  for (int j = j0 + lane; j < n; j += step) {
    const int64_t at = at0 + j;
    if (at >= cap) break;
    // the last ray whose first slot is at or before j (rays without samples
    // share the next ray's first slot and come before it)
    int u = 0;
#pragma unroll
    for (int h = kWave / 2; h > 0; h >>= 1)
      if (first[wid][u + h] <= j) u += h;
    int q = j - first[wid][u], k = 0;
    const uint64_t *mr = masks + (r0 + u) * nw;
    uint64_t m = mr[0];
    for (int c = __popcll(m); q >= c; c = __popcll(m)) {  // the word that holds the q-th kept step
      q -= c;
      k += kWave;
      m = mr[k / kWave];
    }
    k += select_bit64(m, q);
    const float o[3] = {in[wid][0][u], in[wid][1][u], in[wid][2][u]};
    const float d[3] = {in[wid][3][u], in[wid][4][u], in[wid][5][u]};
    float t, x[3];
    sample_pos(o, d, in[wid][6][u], in[wid][7][u], k, &t, x);
    xs[at] = x[0];
    xs[cap + at] = x[1];
    xs[2 * cap + at] = x[2];
    ts[at] = t;
    ray_id[at] = (int32_t)(r0 + u);
  }
}

}  // namespace

// Workspace: block totals, chunk totals, keep masks [R][ceil(max_steps/64)]
// and entry distances [R], each slice 256-byte aligned.  Its size never falls
// as R or max_steps grows: a workspace for the largest call of a pool serves
// the smaller ones.  Block totals: one for four rays below kAnyManyRays, from
// there on no fewer, and at least one for 16 rays (one for kBlock would do).
struct MarchWs {
  int64_t *block_sum, *chunk_sum;
  uint64_t *masks;
  float *tn;
  size_t bytes;
};

static MarchWs march_ws(void *base, int64_t R, int32_t max_steps) {
  const int64_t Rp = R > 0 ? R : 1, few = Rp < kAnyManyRays ? Rp : kAnyManyRays - 1;
  const int64_t per_wave = ceil_div(max_steps <= kManySteps ? few : Rp, kWavesPerBlock), rest = ceil_div(Rp, 16);
  const int64_t nblk = per_wave > rest ? per_wave : rest;
  const int64_t nw = ceil_div(max_steps > 0 ? max_steps : 1, kWave);
  char *p = (char *)base;
  MarchWs w;
  size_t o = 0;
  w.block_sum = (int64_t *)(p + o);
  o += align256(sizeof(int64_t) * (size_t)nblk);
  w.chunk_sum = (int64_t *)(p + o);
  o += align256(sizeof(int64_t) * (size_t)ceil_div(nblk, kScanChunk));
  w.masks = (uint64_t *)(p + o);
  o += align256(sizeof(uint64_t) * (size_t)(Rp * nw));
  w.tn = (float *)(p + o);
  o += align256(sizeof(float) * (size_t)Rp);
  w.bytes = o;
  return w;
}

extern "C" size_t ia355_march_workspace_size(int64_t R, int32_t max_steps) {
  if (R < 0 || max_steps < 0) return 0;
  return march_ws(nullptr, R, max_steps).bytes;
}

extern "C" int32_t ia355_occgrid_march(const float *rays_o, const float *rays_d, int64_t R, const uint32_t *occ_bits,
                                       int32_t G, const float *aabb, float dt, int32_t n_per_ray, int32_t max_steps,
                                       float *xs, float *ts, int32_t *ray_id, int64_t cap, int64_t *ray_off,
                                       int32_t *ray_cnt, float *ray_dt, int64_t *n_samples, int64_t *n_required,
                                       void *ws, size_t ws_bytes, ia355_stream_t stream) {
  if (R < 0 || !aabb || max_steps < 0 || cap < 0) return IA355_ERR_INVALID_ARG;
  if (!ray_off || !n_samples) return IA355_ERR_INVALID_ARG;
  if (R > 0 && (!rays_o || !rays_d || !ray_cnt || !ray_dt)) return IA355_ERR_INVALID_ARG;
  if (cap > 0 && (!xs || !ts || !ray_id)) return IA355_ERR_INVALID_ARG;
  if (occ_bits && (G <= 0 || G > 2048)) return IA355_ERR_INVALID_ARG;
  if (n_per_ray <= 0 && !(dt > 0.0f)) return IA355_ERR_INVALID_ARG;
  if ((int64_t)cap * 3 < cap) return IA355_ERR_INVALID_ARG;
  if (!ws || ws_bytes < ia355_march_workspace_size(R, max_steps)) return IA355_ERR_WORKSPACE;
  Box box;
  bool pow2;
  if (!make_box(aabb, &box, &pow2)) return IA355_ERR_INVALID_ARG;
  hipStream_t s = as_stream(stream);
  const bool many = many_rays(R, max_steps, aabb, dt, n_per_ray);
  const int64_t nblk = ceil_div(R, many ? kBlock : kWavesPerBlock);
  const int64_t nchunk = ceil_div(nblk, kScanChunk);
  const int nw = (int)ceil_div(max_steps, kWave);
  const MarchWs mw = march_ws(ws, R, max_steps);
  int64_t *block_sum = mw.block_sum, *chunk_sum = mw.chunk_sum;
  if (R > 0) {
    if (many) {
      const bool zero = box.lo[0] == 0.0f && box.lo[1] == 0.0f && box.lo[2] == 0.0f;
      auto *fn = !occ_bits ? march_count_many<kGeneral, false>  // without a grid no cell is looked up
                 : !pow2   ? march_count_many<kGeneral, true>
                 : zero    ? march_count_many<kPow2AtZero, true>
                           : march_count_many<kPow2, true>;
      fn<<<(unsigned)nblk, kBlock, 0, s>>>(rays_o, rays_d, R, reinterpret_cast<const uint8_t *>(occ_bits), G, box, dt,
                                           n_per_ray, max_steps, ray_off, ray_cnt, ray_dt, block_sum, mw.masks, nw,
                                           mw.tn);
    } else if (pow2)
      march_count<true><<<(unsigned)nblk, kBlock, 0, s>>>(rays_o, rays_d, R, occ_bits, G, box, dt, n_per_ray,
                                                          max_steps, ray_off, ray_cnt, ray_dt, block_sum, mw.masks, nw,
                                                          mw.tn);
    else
      march_count<false><<<(unsigned)nblk, kBlock, 0, s>>>(rays_o, rays_d, R, occ_bits, G, box, dt, n_per_ray,
                                                           max_steps, ray_off, ray_cnt, ray_dt, block_sum, mw.masks,
                                                           nw, mw.tn);
    auto *scan = nblk <= 1024 ? march_scan_chunk<1> : nblk <= 4096 ? march_scan_chunk<4> : march_scan_chunk<kScanPer>;
    scan<<<(unsigned)nchunk, 1024, 0, s>>>(block_sum, nblk, chunk_sum, ray_off, R, n_samples);
  }
  if (nchunk != 1) march_scan_top<<<1, 1024, 0, s>>>(chunk_sum, nchunk, ray_off, R, n_samples);
  if (R > 0 && cap > 0) {
    if (many)
      march_fill_many<<<dim3((unsigned)nblk, fill_parts(R)), kBlock, 0, s>>>(
          rays_o, rays_d, R, mw.masks, nw, mw.tn, block_sum, chunk_sum, ray_off, ray_cnt, ray_dt, xs, ts, ray_id, cap);
    else
      march_fill<<<(unsigned)nblk, kBlock, 0, s>>>(rays_o, rays_d, R, mw.masks, nw, mw.tn, block_sum, chunk_sum,
                                                   ray_off, ray_dt, xs, ts, ray_id, cap);
  }
  const int32_t st = launch_status();
  if (st != IA355_OK || !n_required) return st;
  // synchronous capacity check, on request only
  int64_t n = 0;
  if (hipMemcpyAsync(&n, n_samples, sizeof n, hipMemcpyDeviceToHost, s) != hipSuccess) return IA355_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return IA355_ERR_HIP;
  *n_required = n;
  return n > cap ? IA355_ERR_CAPACITY : IA355_OK;
}
