// Multiresolution hash encoding (Sec. 3.1, Instant-NGP) forward and backward.
//
// Forward design (gfx950, 8 XCDs with a private 4 MB L2 each):
//  * a lane takes a sample (two in frame-sized calls) and two levels where an
//    XCD serves several: a block's 256 or 512 consecutive samples read their
//    positions once for both, and its gathers stay inside two levels' tables;
//  * workgroups are dispatched round-robin over the 8 XCDs, so block b runs
//    on XCD b % 8, and levels are assigned to XCDs (xcd_level): each XCD's L2
//    caches the tables of two levels at a time (2 x 2 MiB at T = 2^19 in FP16)
//    instead of all sixteen.  With an FP32 table an XCD keeps its levels for
//    the call, with an FP16 one the pairs move on seven times (served_xcd);
//  * the position scaling u = x N_l is split into a rounded product and its
//    exact FMA remainder, so the cell and fraction are accurate to FP32
//    relative precision even at N_l ~ 2000;
//  * features are written level-major [L][S][F]: each block writes one
//    contiguous run a level (coalesced 8-byte / 4-byte stores per lane).
// Backward: the table gradient sorts corner pairs by tile of the table and sums
// each tile in LDS as integers, or, without a workspace, adds FP32 atomics laid
// out so that each wave instruction touches few cache lines (see
// table_grad_kernel); the position gradient has the forward's mapping, a level's
// contributions in a workspace, then their sum in a fixed order (deterministic).
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>

#include "common.h"
#include "hash_dev.h"

using namespace ia355;
using namespace ia355::hsh;

namespace {

constexpr int kFwdBlock = 256;
constexpr int64_t kTwoSampleMin = (int64_t)1 << 22;  // samples (or capacity) from which a lane takes two
// Chunk slots with a device-side count: 1024, and with an FP16 table a quarter
// of what the capacity holds if that is more, at most 4096.  Blocks of one
// chunk, taken in order, keep what runs at a time to neighbouring samples and
// to one or two phases of served_xcd; blocks that loop drift apart.  Past the
// count a slot's eight blocks cost 1.4 ns, as they leave before anything else
// (4 where they first worked out their levels: 5000 points under a capacity of
// 2,332,800 took 12.0 us, 6.4 now; with 1024 slots they take 5.1).  1024, 2048 and 4096 slots, FP16:
// frames of 540 x 540 (9112 chunks of capacity) with 0.88 M samples 305, 300
// and 296 us, with 0.44 M 193, 192 and 200; of 300 x 300 (2813) 123, 125 and
// 129; a training step (4096, 143 in use) 247, 247 and 255.  FP32 steps gain
// nothing (325.1 us with 1024, 325.7 with 4096).
constexpr int64_t kDevSlots = 1024, kDevSlotsMost = 4096;

// Level of a lane's slot t in level group g on XCD x, or -1 (no level).  With
// two levels per lane and at most 16 levels, XCD x serves level x and level
// L - 1 - x (when that is 8 or more): coarse levels, whose samples share
// cells, pair with fine ones, whose gathers are scattered, so every XCD gets
// a similar load and at most one fine table.  Otherwise XCD x serves levels
// x + 8 (kLv g + t).
template <int kLv>
__device__ __forceinline__ int xcd_level(int x, int g, int t, int L) {
  if (kLv == 2 && L <= 2 * kXcd) {
    const int l = t == 0 ? x : L - 1 - x;
    return (t == 0 ? l < L : l >= kXcd) ? l : -1;
  }
  const int l = x + kXcd * (kLv * g + t);
  return l < L ? l : -1;
}

// The XCD whose levels a block serves.  FP16 table: the pairs move on by one
// XCD seven times a call -- the slots in use, which run about in order, are
// eight phases, and in phase p XCD x serves what xcd_level gives for
// (x + p) % 8.  The pairs are not equally dear (of 16 levels from 16 up by
// 1.38 with 2^19 entries, eleven are hashed: some pairs have two scattered levels), and the call
// lasted as long as the dearest: 1,000,003 points 125.5 -> 113.3 us.  An FP32
// level of 2^19 entries fills an XCD's 4 MB L2, and fetching eight of them
// costs what the balance gives (0.4 to 1 % slower over training steps and
// grid updates): it stays.  The FP16 position gradient gains alike (262,143
// points: encode 36 -> 33 us, gradient 41 -> 38 us).
template <typename TT>
__device__ __forceinline__ int served_xcd(int slot, int64_t nslot, int64_t chunks) {
  const uint32_t used = (uint32_t)(chunks < nslot ? chunks : nslot);  // nslot < 2^28
  if (sizeof(TT) != 2 || (uint32_t)slot >= used) return blockIdx.x % kXcd;
  return (blockIdx.x + (uint32_t)slot * kXcd / used) % kXcd;
}

// Block b works on XCD b % 8 on the levels xcd_level gives served_xcd's slots
// t < kLv in level group g = slot % ngroup (slot = b / 8), on chunks of
// 256 kSp samples slot / ngroup, + nslot, + 2 nslot ...  A lane takes kSp
// samples of a chunk (256 apart) and reads each sample's position and bone
// once for its kLv levels; all their corner gathers are in flight together.
template <typename TT, typename FT, int kLv, int kSp>
__global__ void __launch_bounds__(kFwdBlock) encode_kernel(const float *__restrict__ xc, const int16_t *__restrict__ bone,
                                                           int64_t S, const int64_t *__restrict__ S_dev, int64_t ld,
                                                           const TT *__restrict__ table, int L, int log2T, Levels lv,
                                                           Box box, FT *__restrict__ feat, int ngroup) {
  const int slot = blockIdx.x / kXcd;
  const int64_t Sn = count_of(S, S_dev);
  const int64_t nslot = gridDim.x / (kXcd * ngroup);
  constexpr int64_t kSpan = (int64_t)kFwdBlock * kSp;
  if (slot >= ceil_div(Sn, kSpan) * ngroup) return;  // no chunk
  const int xcd = served_xcd<TT>(slot / ngroup, nslot, ceil_div(Sn, kSpan));
  int lev[kLv];
#pragma unroll
  for (int t = 0; t < kLv; ++t) lev[t] = xcd_level<kLv>(xcd, slot % ngroup, t, L);
  if (lev[0] < 0) return;
  const uint32_t T = 1u << log2T;
  for (int64_t chunk = slot / ngroup; chunk * kSpan < Sn; chunk += nslot) {
    int64_t n[kSp];
    float x[kSp][3];
    int bv[kSp];
    bool in[kSp], use[kSp];
    // positions and bones loaded together (one round trip; the bones are
    // tested only after every load is issued)
#pragma unroll
    for (int sp = 0; sp < kSp; ++sp) {
      n[sp] = chunk * kSpan + sp * kFwdBlock + threadIdx.x;
      in[sp] = n[sp] < Sn;
      const int64_t m = in[sp] ? n[sp] : 0;
      x[sp][0] = xc[m];
      x[sp][1] = xc[ld + m];
      x[sp][2] = xc[2 * ld + m];
      bv[sp] = 0;
    }
    if (bone)
#pragma unroll
      for (int sp = 0; sp < kSp; ++sp) bv[sp] = bone[in[sp] ? n[sp] : 0];
#pragma unroll
    for (int sp = 0; sp < kSp; ++sp) use[sp] = in[sp] && bv[sp] >= 0;
    float a[kSp][kLv], b[kSp][kLv];
#pragma unroll
    for (int sp = 0; sp < kSp; ++sp)
#pragma unroll
      for (int t = 0; t < kLv; ++t) a[sp][t] = b[sp][t] = 0.0f;
    // every lane encodes (no branch around the gathers, so all of them are
    // in flight together; any position gives in-range cells); samples
    // without a root then store zeros
#pragma unroll
    for (int sp = 0; sp < kSp; ++sp)
#pragma unroll
      for (int t = 0; t < kLv; ++t) {
        const int level = lev[t];
        if (level >= 0)
          encode_level(x[sp], box, lv.res[level], lv.dense[level], T - 1u, table + (int64_t)level * T * 2, &a[sp][t],
                       &b[sp][t]);
      }
#pragma unroll
    for (int sp = 0; sp < kSp; ++sp)
      if (in[sp])
#pragma unroll
        for (int t = 0; t < kLv; ++t) {
          const int level = lev[t];
          if (level >= 0)
            store_feat2(feat, (int64_t)level * ld + n[sp], use[sp] ? a[sp][t] : 0.0f, use[sp] ? b[sp][t] : 0.0f);
        }
  }
}

struct EncodeArgs {
  const float *xc;
  const int16_t *bone;
  int64_t S;
  const int64_t *S_dev;
  int64_t ld;
  const void *table;
  int L, log2T;
  Levels lv;
  Box box;
  void *feat;
  int ngroup;
};

template <typename TT, typename FT>
void launch_encode(const EncodeArgs &a, int lv_lane, int sp_lane, unsigned g, hipStream_t s) {
  const TT *t = static_cast<const TT *>(a.table);
  FT *f = static_cast<FT *>(a.feat);
  if (lv_lane == 2 && sp_lane == 2)
    encode_kernel<TT, FT, 2, 2><<<g, kFwdBlock, 0, s>>>(a.xc, a.bone, a.S, a.S_dev, a.ld, t, a.L, a.log2T, a.lv, a.box,
                                                        f, a.ngroup);
  else if (lv_lane == 2)
    encode_kernel<TT, FT, 2, 1><<<g, kFwdBlock, 0, s>>>(a.xc, a.bone, a.S, a.S_dev, a.ld, t, a.L, a.log2T, a.lv, a.box,
                                                        f, a.ngroup);
  else
    encode_kernel<TT, FT, 1, 1><<<g, kFwdBlock, 0, s>>>(a.xc, a.bone, a.S, a.S_dev, a.ld, t, a.L, a.log2T, a.lv, a.box,
                                                        f, a.ngroup);
}

// Position gradient dL/dx = sum_l sum_c (grad w_c) (theta_c . dL/dfeat_l),
// in two kernels.  The first has the forward's mapping (block b on XCD
// b % 8, the levels xcd_level gives served_xcd's, one lane per sample): every sample of a
// level is served by one XCD's L2, so cells shared by samples are fetched
// once rather than once per XCD; it writes each level's contribution to a
// workspace part [L][3][S].  The second sums the levels in a fixed order.
constexpr int kBwdBlock = 256;
constexpr int kBwdMaxLevels = 16;  // the backward's level limit
// Wave priority: beside the table gradient of a training step the position
// gradient is the longer chain, and its waves come first where they share a
// SIMD with the sort's (captured step of 8,192 rays: 332 us without, 327 so,
// 330 with the first kernel alone; the moments after it are no faster for it).
constexpr int kXgradPrio = 2;

template <typename TT, int kLv>
__global__ void __launch_bounds__(kBwdBlock) xgrad_level_kernel(
    const float *__restrict__ gfeat, const float *__restrict__ xc, const int16_t *__restrict__ bone, int64_t S,
    const int64_t *__restrict__ S_dev, int64_t ld, const TT *__restrict__ table, int L, int log2T, Levels lv, Box box,
    float *__restrict__ part, int ngroup) {
  __builtin_amdgcn_s_setprio(kXgradPrio);
  // the encode's mapping: kLv levels (b % 8) + 8 (kLv g + t) per lane
  const int slot = blockIdx.x / kXcd;
  const int64_t Sn = count_of(S, S_dev);
  const int64_t nslot = gridDim.x / (kXcd * ngroup);
  if (slot >= ceil_div(Sn, (int64_t)kBwdBlock) * ngroup) return;  // no chunk
  const int xcd = served_xcd<TT>(slot / ngroup, nslot, ceil_div(Sn, (int64_t)kBwdBlock));
  int lev[kLv];
#pragma unroll
  for (int t = 0; t < kLv; ++t) lev[t] = xcd_level<kLv>(xcd, slot % ngroup, t, L);
  if (lev[0] < 0) return;
  const uint32_t T = 1u << log2T;
  for (int64_t chunk = slot / ngroup; chunk * kBwdBlock < Sn; chunk += nslot) {
    const int64_t n = chunk * kBwdBlock + threadIdx.x;
    if (n >= Sn) break;
    float gx[kLv][3];
    float2 g[kLv];
    // position, incoming gradients and bone loaded together (one round trip)
    const float x[3] = {xc[n], xc[ld + n], xc[2 * ld + n]};
#pragma unroll
    for (int t = 0; t < kLv; ++t) {
      const int level = lev[t];
      g[t] = level >= 0 ? reinterpret_cast<const float2 *>(gfeat)[(int64_t)level * ld + n] : make_float2(0.0f, 0.0f);
      gx[t][0] = gx[t][1] = gx[t][2] = 0.0f;
    }
    if (!bone || bone[n] >= 0) {
      // every level's gathers first, then the sums (a missing second level
      // repeats the first with a zero gradient and is not stored)
      Corners c[kLv];
      float2 vv[kLv][8];
#pragma unroll
      for (int t = 0; t < kLv; ++t) {
        const int level = lev[t] >= 0 ? lev[t] : lev[0];
        level_cell(x, box, lv.res[level], lv.dense[level], T - 1u, c[t], true);
        gather8(table + (int64_t)level * T * 2, c[t], vv[t]);
      }
#pragma unroll
      for (int t = 0; t < kLv; ++t)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float d = vv[t][k].x * g[t].x + vv[t][k].y * g[t].y;
          gx[t][0] += c[t].dw[k][0] * d;
          gx[t][1] += c[t].dw[k][1] * d;
          gx[t][2] += c[t].dw[k][2] * d;
        }
    }
#pragma unroll
    for (int t = 0; t < kLv; ++t) {
      const int level = lev[t];
      if (level < 0) continue;
      float *pl = part + (int64_t)level * 3 * S;
      pl[n] = gx[t][0];
      pl[S + n] = gx[t][1];
      pl[2 * S + n] = gx[t][2];
    }
  }
}

template <typename TT>
void launch_xgrad(int lv_lane, unsigned blocks, hipStream_t s, const float *gfeat, const float *xc,
                  const int16_t *bone, int64_t S, const int64_t *S_dev, int64_t ld, const void *table, int L, int log2T,
                  const Levels &lv, const Box &box, float *part, int ngroup) {
  const TT *t = static_cast<const TT *>(table);
  if (lv_lane == 2)
    xgrad_level_kernel<TT, 2><<<blocks, kBwdBlock, 0, s>>>(gfeat, xc, bone, S, S_dev, ld, t, L, log2T, lv, box, part,
                                                           ngroup);
  else
    xgrad_level_kernel<TT, 1><<<blocks, kBwdBlock, 0, s>>>(gfeat, xc, bone, S, S_dev, ld, t, L, log2T, lv, box, part,
                                                           ngroup);
}

__global__ void __launch_bounds__(kBwdBlock) xgrad_sum_kernel(const float *__restrict__ part, int64_t S,
                                                              const int64_t *__restrict__ S_dev, int L, int64_t ld,
                                                              float *__restrict__ gxc) {
  __builtin_amdgcn_s_setprio(kXgradPrio);
  const int64_t Sn = count_of(S, S_dev);
  for (int64_t n = (int64_t)blockIdx.x * kBwdBlock + threadIdx.x; n < Sn; n += (int64_t)gridDim.x * kBwdBlock) {
    // all loads first (independent addresses), then the sums in level order
    float v[kBwdMaxLevels][3];
#pragma unroll
    for (int l = 0; l < kBwdMaxLevels; ++l)
#pragma unroll
      for (int a = 0; a < 3; ++a) v[l][a] = l < L ? part[((int64_t)l * 3 + a) * S + n] : 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      float acc = 0.0f;
#pragma unroll
      for (int l = 0; l < kBwdMaxLevels; ++l)
        if (l < L) acc += v[l][a];
      gxc[a * ld + n] = acc;
    }
  }
}

// Table gradient with coalesced atomics.  FP32 atomics to random addresses
// are limited by L2 requests (one per touched cache line per instruction),
// not by the number of floats added, so the mapping packs updates that
// share lines into the same wave instruction: 16 lanes per (level, sample)
// item, lane = 2 * corner + feature.  The two features of a corner are
// adjacent floats and x-neighbouring corners are adjacent entries (dense
// levels) or differ only in low bits (hashed levels, x prime = 1), so the
// 16 updates of an item touch about four lines.  Items are level-major, so
// the four items of a wave are consecutive samples of one level and share
// lines on the coarse levels as well.
constexpr int kTgBlock = 256;
constexpr int kTgMaxGrid = 1024;      // 4 blocks per CU
constexpr int kTgDenseMaxGrid = 512;  // 2 blocks per CU

__global__ void __launch_bounds__(kTgBlock) table_grad_kernel(const float *__restrict__ gfeat,
                                                             const float *__restrict__ xc,
                                                             const int16_t *__restrict__ bone, int64_t S,
                                                             const int64_t *__restrict__ S_dev, int64_t ld, int l0,
                                                             int L, int log2T, Levels lv, Box box,
                                                             float *__restrict__ gtable) {
  const int64_t Sn = count_of(S, S_dev);
  const int64_t items = (int64_t)(L - l0) * Sn;
  const int sub = (int)(threadIdx.x & 15), k = sub >> 1, f = sub & 1;
  const uint32_t T = 1u << log2T;
  for (int64_t item = ((int64_t)blockIdx.x * kTgBlock + threadIdx.x) >> 4; item < items;
       item += (int64_t)gridDim.x * (kTgBlock / 16)) {
    const int level = l0 + (int)(item / Sn);
    const int64_t n = item - (int64_t)(level - l0) * Sn;  // 0 <= n < Sn
    if (bone && bone[n] < 0) continue;
    const float x[3] = {xc[n], xc[ld + n], xc[2 * ld + n]};
    // this lane's corner only (a runtime-indexed corner array would live in
    // scratch memory)
    const int N = lv.res[level];
    const CellPos cp = level_pos(x, box, N);
    const uint32_t idx = corner_index(cp, k, N, lv.dense[level] != 0, T - 1u);
    const float g = gfeat[2 * ((int64_t)level * ld + n) + f];
    atomicAdd(gtable + 2 * ((int64_t)level * T + idx) + f, corner_weight(cp, k) * g);
  }
}

// Dense (coarse) levels: many consecutive samples fall in the same cell, so
// the same table entries are hit again and again (atomic contention).  One
// lane per sample (a wave = 64 consecutive samples of one level); for each
// corner the lanes are segmented into runs of equal table index and a
// segmented wave scan sums each run, so only the last lane of a run issues
// the atomic adds.
constexpr int kDgBlock = 256;
constexpr int kAggMaxRes = 32;  // finest resolution handled by run aggregation

__global__ void __launch_bounds__(kDgBlock) table_grad_dense_kernel(const float *__restrict__ gfeat,
                                                                   const float *__restrict__ xc,
                                                                   const int16_t *__restrict__ bone, int64_t S,
                                                                   const int64_t *__restrict__ S_dev, int64_t ld,
                                                                   int ndense, int log2T, Levels lv, Box box,
                                                                   float *__restrict__ gtable) {
  const int64_t Sn = count_of(S, S_dev);
  const int64_t chunks = ceil_div(Sn, kDgBlock);
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t T = 1u << log2T;
  // one (level, chunk) pair per block and step; the whole wave takes part
  // in the scans below
  for (int64_t p = blockIdx.x; p < (int64_t)ndense * chunks; p += gridDim.x) {
    const int level = (int)(p / chunks);
    const int64_t n = (p % chunks) * kDgBlock + threadIdx.x;
    const bool act = n < Sn && (!bone || bone[n] >= 0);
    Corners c;
    float2 g = make_float2(0.0f, 0.0f);
    if (act) {
      const float x[3] = {xc[n], xc[ld + n], xc[2 * ld + n]};
      level_cell(x, box, lv.res[level], true, T - 1u, c, false);
      g = reinterpret_cast<const float2 *>(gfeat)[(int64_t)level * ld + n];
    }
    float *gl = gtable + (int64_t)level * T * 2;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int key = act ? (int)c.idx[k] : -1 - lane;  // inactive lanes: unique keys, no atomics
      float v0 = act ? c.w[k] * g.x : 0.0f, v1 = act ? c.w[k] * g.y : 0.0f;
      const int prev = __shfl_up(key, 1, kWave);
      int hs = (lane == 0 || prev != key) ? lane : 0;  // run head index
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(hs, o, kWave);
        if (lane >= o) hs = max(hs, t);
      }
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const float t0 = __shfl_up(v0, o, kWave), t1 = __shfl_up(v1, o, kWave);
        if (lane - o >= hs) {
          v0 += t0;
          v1 += t1;
        }
      }
      const int next = __shfl_down(key, 1, kWave);
      if ((lane == kWave - 1 || next != key) && key >= 0) {
        atomicAdd(gl + 2 * key, v0);
        atomicAdd(gl + 2 * key + 1, v1);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Table gradient without global atomics (binned).  Each level's table is cut
// into tiles of E = 2^tb entries (2 E 8-byte sums fit in LDS); a corner update
// (entry, w_c dL/dfeat_l) belongs to the tile of its entry.  Three passes:
//  1. sort: a workgroup takes one level and kSortChunk samples, counts its
//     updates per tile in LDS (keeping each update's rank in a register),
//     scans the counts and writes its updates in tile order into the chunk's
//     own part of the workspace, and each tile's run, with the largest exponent
//     of its values, into the run table.  A chunk's part is sized for its
//     samples, so no pass has to agree on offsets across workgroups.
//  2. plan: from the run table, a work item for each tile with records, or
//     several, by chunks, for one with many (coarse levels, whose samples
//     crowd on the subject).
//  3. accumulate: a workgroup takes an item at a time, sums its runs into an
//     LDS copy of the tile and writes it with plain vector stores, or adds its
//     nonzero entries with global atomics where several share the tile.
// The work items depend on the positions alone, so a first call may make them
// before the gradients are known; the second then sorts and accumulates.
// The two x-neighbouring corners of a cell are adjacent entries or differ in
// their low index bits (the x prime is 1), so they nearly always fall in one
// tile and travel as one 16-byte record: the two features' (w_y w_z) dL/dfeat,
// the x fraction and both entries.  Corners of a pair that a tile boundary
// separates are 12-byte records at the end of the chunk's part; a sample's
// eight updates take at most 96 bytes either way.
// The LDS sums are 64-bit fixed point, added exactly: LDS float atomic adds run at
// about a sixteenth of the rate of integer ones on gfx950, so each work item
// scales its values by a power of two 2^s chosen from its largest |value| m
// (no overflow), adds them as integers and converts each entry back once.
// Each value is rounded to the quantum 2^-s <= m 2^-46, so an entry's error is
// at most (its values) x m 2^-47 plus one FP32 rounding, and one more per
// addition to the table where items share the tile: an absolute bound relative
// to the item's largest value.  An entry near m is as accurate as FP32 adds
// leave it or better; one far below m (under about m 2^-24) is less accurate
// than FP32 adds, and a value below m 2^-48 rounds to zero.  Integer addition
// is associative, so a tile summed by one workgroup (any with 8192 records or
// fewer) does not depend on the order of its records.
// The traffic is the records (64 bytes per sample and level, written once and
// read once) and one pass over the table slice.
// 16 levels of 2^19 entries, field gradients (traced: sort, plan,
// accumulate): 19 + 9 + 36 us for 36,503 samples, 100 + 13 + 115 us for
// 262,143.  With a scale, a conversion and a clear of the tile for each window
// of at most 4096 records, whose maximum the workgroup found first: 17 + 10 +
// 43 and 101 + 15 + 146 us.  Counting, scanning and placing 12-byte single
// records across all workgroups took six passes, 85 and 422 us: four of them
// only to agree on offsets, and every 4096 records flushed a tile with global
// atomics.  A fixed share of a level's tiles per item in place of the plan left
// the accumulate pass 62 and 243 us (the largest items ran on alone for half
// of it).
constexpr int kSortBlock = 320;
constexpr int kSortPer = 4;                        // samples per thread
constexpr int kSortChunk = kSortBlock * kSortPer;  // at 128 tiles a hashed level's runs average 40 pairs
constexpr int kSampleBytes = 96;   // record space of one sample and level
constexpr int kMaxBins = 16384;    // tiles over all levels
constexpr int kTileLog2Max = 12;   // 4096 entries x 2 x 8 B = 64 KB of LDS
constexpr int kAccBlock = 512;
constexpr int kAccWaves = kAccBlock / kWave;
constexpr int kAccPer = 8;         // records per thread and window
constexpr int kRunWaves = 4;       // waves that load a batch's runs, one per lane
constexpr int kAccRuns = kRunWaves * kWave;
// Records of a work item at least, where a tile has more (each item of a shared
// tile costs an addition per entry it holds: with 4096, 36,503 random points in
// tables of 2^12 to 2^17 took 10 to 28 us more of 50 to 90, on a surface and
// 2^19 entries 3 us less of 65), and at most, but for its last chunk's.
constexpr uint32_t kAccTarget = 8192, kAccMost = 32768;
constexpr int kPlanBlock = 1024;
constexpr uint32_t kNoItem = 0xffffffffu;
constexpr int kAccWr = (1 << (kTileLog2Max - 1)) / kAccBlock;  // float4 of a tile per thread
constexpr int kAccSums = 2 << kTileLog2Max;
constexpr int kAccMaxGrid = 512;   // two workgroups per CU by LDS
static_assert(4 * kSortChunk < 1 << 13 && 8 * kSortChunk < 1 << 14, "run places");
static_assert(kAccMost + 8 * kSortChunk < 1 << 16, "fixed-point head room");

struct BinGeom {
  int tb;        // log2 entries per tile
  int tpl_log2;  // log2 tiles per level
  int64_t chunks;  // sort chunks of the capacity
};

inline bool bin_geom(int nl, int64_t S, int log2T, BinGeom *g) {
  if (nl <= 0 || S < 0 || log2T < 1 || log2T > 30) return false;
  g->tb = log2T < kTileLog2Max ? log2T : kTileLog2Max;
  g->tpl_log2 = log2T - g->tb;
  if (((int64_t)nl << g->tpl_log2) > kMaxBins) return false;
  g->chunks = ceil_div(S > 0 ? S : 1, (int64_t)kSortChunk);
  return (int64_t)nl * S * 8 < 0xffffffffLL;
}

// runs[level][tile][chunk], see pack_run; rec: chunk c of level lr has the
// bytes from (lr S + c kSortChunk) 96, pair records upwards from its start,
// single records downwards from its end.
struct BinQueue {
  uint32_t next;          // items that the accumulate pass took from the queue
  uint32_t split, whole;  // work items of tiles that several share, of whole tiles
};

// A run: its first pair record and their number, the same of its single
// records, the largest exponent field of its finite values, and whether its
// chunk holds a NaN or an infinity on this level.
__device__ __forceinline__ uint2 pack_run(uint32_t p0, uint32_t pn, uint32_t s0, uint32_t sn, uint32_t ex,
                                          uint32_t odd) {
  return make_uint2(p0 | pn << 13 | (ex & 63u) << 26, s0 | sn << 14 | (ex >> 6) << 28 | odd << 30);
}
__device__ __forceinline__ uint32_t run_pairs(const uint2 &q) { return (q.x >> 13) & 0x1fffu; }
__device__ __forceinline__ uint32_t run_singles(const uint2 &q) { return (q.y >> 14) & 0x3fffu; }
__device__ __forceinline__ uint32_t run_exponent(const uint2 &q) { return q.x >> 26 | ((q.y >> 28) & 3u) << 6; }
__device__ __forceinline__ bool run_odd(const uint2 &q) { return (q.y >> 30) != 0u; }

// A work item of the accumulate pass: a range of chunks of a tile.
struct AccItem {
  uint32_t bin;     // level << tpl_log2 | tile
  uint32_t c0, c1;  // chunks
  uint32_t split;   // summed with atomics
};

struct BinWs {
  BinQueue *queue;
  AccItem *items;  // shared tiles' from the start on, whole tiles' from the end down
  int64_t cap;     // of items: a tile of n records has at most n / kAccTarget + 1
  uint8_t *shared;  // per tile: no whole item, so an overwrite clears it before the accumulate pass
  uint2 *runs;
  char *rec;
  size_t bytes;
};

inline BinWs bin_ws(int nl, int64_t S, const BinGeom &g, void *base) {
  BinWs w;
  char *p = (char *)base;
  size_t o = 0;
  w.queue = (BinQueue *)(p + o);
  o += 256;
  w.items = (AccItem *)(p + o);
  w.cap = ((int64_t)nl << g.tpl_log2) + (int64_t)nl * S * 8 / kAccTarget;
  o += align256(sizeof(AccItem) * (size_t)w.cap);
  w.shared = (uint8_t *)(p + o);
  o += align256((size_t)nl << g.tpl_log2);
  w.rec = p + o;
  o += align256((size_t)kSampleBytes * (size_t)nl * (size_t)(S > 0 ? S : 1));
  w.runs = (uint2 *)(p + o);  // after the records: a single record is loaded with the four bytes behind it
  o += align256(sizeof(uint2) * (((size_t)nl * (size_t)g.chunks) << g.tpl_log2));
  w.bytes = o;
  return w;
}

// Exclusive scan of one value per thread over a block of kThreads; *total
// gets the block's sum (the same in every thread).
template <int kThreads>
__device__ __forceinline__ uint32_t block_scan_u32(uint32_t v, uint32_t *wsum, uint32_t *total) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const uint32_t incl = (uint32_t)wave_incl_scan((int)v);
  if (lane == kWave - 1) wsum[wid] = incl;
  __syncthreads();
  uint32_t base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) {
    base += w < wid ? wsum[w] : 0u;
    all += wsum[w];
  }
  __syncthreads();
  *total = all;
  return base + incl - v;
}

// Adds 1 to the LDS counter c[bin[k]].x for each lane with act[k], k < 4, and
// gives the counter's value before the lane's own add.  few: the wave's bins
// are likely one or two (dense levels: neighbouring samples); the lanes that
// share the first lane's bin then make one add of their number, instead of
// that many serialised on one LDS address.
__device__ __forceinline__ void wave_reserve4(uint2 *c, const int bin[4], const bool act[4], bool few,
                                              uint32_t rank[4]) {
  if (!few) {
#pragma unroll
    for (int k = 0; k < 4; ++k) rank[k] = act[k] ? atomicAdd(&c[bin[k]].x, 1u) : 0u;
    return;
  }
  const int lane = threadIdx.x & (kWave - 1);
  uint64_t same[4];
  uint32_t own[4], base[4];
  int first[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {  // every add in flight before the first is used
    const uint64_t am = __ballot(act[k]);
    first[k] = am ? __ffsll((unsigned long long)am) - 1 : 0;
    const int b0 = __builtin_amdgcn_readlane(bin[k], first[k]);
    same[k] = __ballot(act[k] && bin[k] == b0);
    const bool lead = lane == first[k] && same[k] != 0ull, alone = act[k] && bin[k] != b0;
    base[k] = own[k] = 0u;
    if (lead || alone) own[k] = atomicAdd(&c[bin[k]].x, lead ? (uint32_t)__popcll(same[k]) : 1u);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    base[k] = (uint32_t)__builtin_amdgcn_readlane((int)own[k], first[k]);
    const bool mine = (same[k] >> lane) & 1ull;
    rank[k] = mine ? base[k] + (uint32_t)__popcll(same[k] & ((1ull << lane) - 1ull)) : own[k];
  }
}

struct SingleRec {
  float a, b;
  uint32_t entry;
};

// Single record i of the chunk whose part ends at `end`.
__device__ __forceinline__ SingleRec *single_at(char *end, uint32_t i) {
  return reinterpret_cast<SingleRec *>(end) - 1 - i;
}

// A store whose line is not needed in the cache again.
__device__ __forceinline__ void store_once(float4 *p, const float4 &v) {
  __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4 *>(p));
}

// Zeroes a tile with `threads` threads.
__device__ __forceinline__ void clear_tile(float *gtable, uint32_t bin, int l0, int log2T, int tb, int thread,
                                           int threads) {
  float4 *dst = reinterpret_cast<float4 *>(gtable + ((((int64_t)l0 << log2T) + ((int64_t)bin << tb)) << 1));
  for (int i = thread; i < 1 << (tb - 1); i += threads) store_once(dst + i, make_float4(0.0f, 0.0f, 0.0f, 0.0f));
}

// |v|, or zero for a NaN or an infinity.
__device__ __forceinline__ float finite_abs(float v) {
  const float a = fabsf(v);
  return a < INFINITY ? a : 0.0f;
}
__device__ __forceinline__ uint32_t exponent_of(float nonnegative) { return __float_as_uint(nonnegative) >> 23; }

// The passes of a call: all of them, those that need only the positions (the
// counts and the work items), or the others.
enum BinPhase { kBinAll, kBinPlan, kBinRest };

template <BinPhase kPhase>
__global__ void __launch_bounds__(kSortBlock, 6) bin_sort_kernel(
    const float *__restrict__ gfeat, const float *__restrict__ xc, const int16_t *__restrict__ bone, int64_t S,
    const int64_t *__restrict__ S_dev, int64_t ld, int l0, int nl, int log2T, int tb, Levels lv, Box box,
    int64_t chunk_cap, BinQueue *__restrict__ queue, uint2 *__restrict__ runs, char *__restrict__ rec,
    const uint8_t *__restrict__ shared, float *__restrict__ gtable) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (kPhase == kBinRest)
      queue->next = 0u;
    else
      *queue = BinQueue{0u, 0u, 0u};
  }
  // per tile: pair records, single records << 16; the largest exponent field
  extern __shared__ uint2 cnt[];
  __shared__ uint32_t wsum[kSortBlock / kWave];
  __shared__ int odd;  // the chunk holds a NaN or an infinity
  const int tpl_log2 = log2T - tb, tiles = 1 << tpl_log2;
  const int lr = blockIdx.x % nl, level = l0 + lr;
  const int N = lv.res[level];
  const bool dense = lv.dense[level] != 0;
  const uint32_t Tmask = (1u << log2T) - 1u, emask = (1u << tb) - 1u;
  const int64_t Sn = count_of(S, S_dev);
  const int64_t chunks = ceil_div(Sn, (int64_t)kSortChunk);
  // Consecutive lanes take consecutive samples, but on dense levels samples a
  // sixty-fourth of the chunk apart: those of a ray share coarse cells, and
  // their records, which follow in lane order, would meet on one LDS address
  // in the accumulate pass.
  const int sample0 = dense ? (int)(threadIdx.x % kWave) * (kSortChunk / kWave) + (int)(threadIdx.x / kWave) * kSortPer
                            : (int)threadIdx.x;
  const int sstep = dense ? 1 : kSortBlock;
  for (int64_t c = blockIdx.x / nl; c < chunks; c += gridDim.x / nl) {
    for (int i = threadIdx.x; i < tiles; i += kSortBlock) cnt[i] = make_uint2(0u, 0u);
    if (threadIdx.x == 0) odd = 0;
    float x[kSortPer][3];
    bool act[kSortPer];
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      const int64_t n = c * kSortChunk + sample0 + j * sstep, q = n < Sn ? n : 0;
      x[j][0] = xc[q];
      x[j][1] = xc[ld + q];
      x[j][2] = xc[2 * ld + q];
      act[j] = n < Sn && (!bone || bone[q] >= 0);
    }
    __syncthreads();
    // rank of each pair within its tile's run, 16 bits each
    uint2 rank[kSortPer];
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      const CellPos p = level_pos(x[j], box, N);
      int t0[4], t1[4];
      bool pair[4];
      uint32_t r[4], idx[8];
      cell_indices(p, N, dense, Tmask, idx);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        t0[k] = (int)(idx[2 * k] >> tb);
        t1[k] = (int)(idx[2 * k + 1] >> tb);
        pair[k] = act[j] && t0[k] == t1[k];
      }
      wave_reserve4(cnt, t0, pair, dense, r);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (act[j] && !pair[k]) {
          atomicAdd(&cnt[t0[k]].x, 1u << 16);
          atomicAdd(&cnt[t1[k]].x, 1u << 16);
        }
      rank[j] = make_uint2((r[0] & 0xffffu) | r[1] << 16, (r[2] & 0xffffu) | r[3] << 16);
    }
    __syncthreads();
    if (kPhase == kBinPlan) {
      for (int i = threadIdx.x; i < tiles; i += kSortBlock)
        runs[(((int64_t)lr << tpl_log2) + i) * chunk_cap + c] =
            pack_run(0u, cnt[i].x & 0xffffu, 0u, cnt[i].x >> 16, 0u, 0u);
      __syncthreads();  // the counters are cleared for the next chunk
      continue;
    }
    // counts -> offsets, in place
    uint32_t carry = 0;
    for (int b0 = 0; b0 < tiles; b0 += kSortBlock) {
      const int i = b0 + threadIdx.x;
      const uint32_t v = i < tiles ? cnt[i].x : 0u;
      uint32_t total;
      const uint32_t off = carry + block_scan_u32<kSortBlock>(v, wsum, &total);  // the halves do not overflow
      if (i < tiles) cnt[i].x = off;
      carry += total;
    }
    __syncthreads();
    char *region = rec + ((int64_t)lr * S + c * kSortChunk) * kSampleBytes;
    uint4 *pairs = reinterpret_cast<uint4 *>(region);
    char *end = region + (Sn - c * kSortChunk < kSortChunk ? Sn - c * kSortChunk : kSortChunk) * kSampleBytes;
#pragma unroll
    for (int j = 0; j < kSortPer; ++j) {
      if (!act[j]) continue;
      // the cell is found again: kept for four samples since the count, it
      // would cost a hundred registers
      asm volatile("" : "+v"(x[j][0]), "+v"(x[j][1]), "+v"(x[j][2]));
      const float2 g = reinterpret_cast<const float2 *>(
          gfeat)[(int64_t)level * ld + c * kSortChunk + sample0 + j * sstep];
      const float top = fmaxf(finite_abs(g.x), finite_abs(g.y));
      if (!(fabsf(g.x) + fabsf(g.y) < INFINITY)) odd = 1;
      const CellPos p = level_pos(x[j], box, N);
      const float w0 = 1.0f - p.f[0], w1 = p.f[0], wx = fmaxf(w0, w1);
      uint32_t idx[8];
      cell_indices(p, N, dense, Tmask, idx);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i0 = idx[2 * k], i1 = idx[2 * k + 1];
        const float wyz = ((k & 1) ? p.f[1] : 1.0f - p.f[1]) * ((k & 2) ? p.f[2] : 1.0f - p.f[2]);
        const float a = wyz * g.x, b = wyz * g.y;
        const uint32_t t0 = i0 >> tb, t1 = i1 >> tb, e0 = i0 & emask, e1 = i1 & emask;
        // few of a tile's values raise its largest exponent: a read and a
        // compare for most
        if (t0 == t1) {
          const uint32_t r = ((k & 2 ? rank[j].y : rank[j].x) >> (k & 1 ? 16 : 0)) & 0xffffu;
          const uint2 q = cnt[t0];
          const uint32_t ex = exponent_of(wx * (wyz * top));  // the largest value's (rounding is monotonic)
          if (ex > q.y) atomicMax(&cnt[t0].y, ex);
          pairs[(q.x & 0xffffu) + r] =
              make_uint4(__float_as_uint(a), __float_as_uint(b), __float_as_uint(w1), e0 | e1 << 16);
        } else {  // the singles' next places are counted in the high halves
          atomicMax(&cnt[t0].y, exponent_of(w0 * (wyz * top)));
          atomicMax(&cnt[t1].y, exponent_of(w1 * (wyz * top)));
          *single_at(end, atomicAdd(&cnt[t0].x, 1u << 16) >> 16) = SingleRec{w0 * a, w0 * b, e0};
          *single_at(end, atomicAdd(&cnt[t1].x, 1u << 16) >> 16) = SingleRec{w1 * a, w1 * b, e1};
        }
      }
    }
    __syncthreads();
    // the run table; a tile's single records end where the next one's begin
    for (int i = threadIdx.x; i < tiles; i += kSortBlock) {
      const uint32_t p0 = cnt[i].x & 0xffffu, p1 = (i + 1 < tiles ? cnt[i + 1].x : carry) & 0xffffu;
      const uint32_t s0 = i ? cnt[i - 1].x >> 16 : 0u, s1 = cnt[i].x >> 16;
      runs[(((int64_t)lr << tpl_log2) + i) * chunk_cap + c] =
          pack_run(p0, p1 - p0, s0, s1 - s0, cnt[i].y, (uint32_t)odd);
    }
    __syncthreads();  // the counters are cleared for the next chunk
  }
  if (kPhase == kBinRest && gtable)  // overwriting: what the plan pass clears otherwise
    for (uint32_t bin = blockIdx.x; bin < (uint32_t)nl << (log2T - tb); bin += gridDim.x)
      if (shared[bin]) clear_tile(gtable, bin, l0, log2T, tb, threadIdx.x, kSortBlock);
}

// v scale rounded to an integer (ties to even), as two's complement bits
// (|v| scale < 2^50): the sum with 1.5 2^52 has it in its low bits.
__device__ __forceinline__ unsigned long long to_fixed(float v, double scale) {
  const double magic = 6755399441055744.0;
  return (unsigned long long)(__double_as_longlong(fma((double)v, scale, magic)) - __double_as_longlong(magic));
}

// A fixed-point sum back to FP32 (one rounding); inv: 1 / scale.
__device__ __forceinline__ float from_fixed(unsigned long long a, double inv) { return (float)((double)(long long)a * inv); }

// Sixteen bytes at a multiple of four.
__device__ __forceinline__ uint4 load16(const char *p) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
  const u4 v = *reinterpret_cast<const u4 *>(p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// The two features of a record's first and second entry (raw: a, b, x
// fraction, entries), or of a single record's entry (a, b, entry; kind 1).
__device__ __forceinline__ float4 values(const uint4 &raw, int kind) {
  const float x = kind ? 0.0f : __uint_as_float(raw.z), a = __uint_as_float(raw.x), b = __uint_as_float(raw.y);
  return make_float4((1.0f - x) * a, (1.0f - x) * b, x * a, x * b);
}

// The work items of the accumulate pass, a wave per tile.  A tile without
// records is cleared here when overwriting, and one with more than `target`
// is split at the chunks where about as many are reached; its workgroups add
// to the table with atomics, so it is cleared as well.  The items so hold at
// most target records and a chunk's, whatever the samples crowd on.  Reads the
// run table once or twice (0.5 MB for 36,503 samples, 3.4 MB for 262,143).
__global__ void __launch_bounds__(kPlanBlock) bin_plan_kernel(const uint2 *__restrict__ runs, int64_t S,
                                                              const int64_t *__restrict__ S_dev, int64_t chunk_cap,
                                                              int l0, int nl, int log2T, int tb, int64_t cap,
                                                              BinQueue *__restrict__ queue,
                                                              AccItem *__restrict__ items,
                                                              uint8_t *__restrict__ shared,
                                                              float *__restrict__ clear) {
  __shared__ uint32_t wholes, first_whole;
  const int lane = threadIdx.x & (kWave - 1), tpl_log2 = log2T - tb;
  const uint32_t bin =
      __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kPlanBlock / kWave) + threadIdx.x / kWave));
  const bool live = bin < (uint32_t)nl << tpl_log2;
  if (threadIdx.x == 0) wholes = 0u;
  const uint32_t Sn = (uint32_t)count_of(S, S_dev), chunks = (Sn + kSortChunk - 1) / kSortChunk;
  const uint2 *run = runs + (int64_t)bin * chunk_cap;
  uint32_t total = 0;
#pragma unroll 4
  for (uint32_t c = lane; live && c < chunks; c += kWave) {
    const uint2 q = run[c];
    total += run_pairs(q) + run_singles(q);
  }
  total = (uint32_t)__builtin_amdgcn_readlane(wave_incl_scan((int)total), kWave - 1);
  // half of what a resident workgroup would get of a level mix without empty
  // tiles, so the largest items do not outlast the others
  const uint32_t even = 4u * (uint32_t)nl * Sn / (2u * kAccMaxGrid);  // 8 L S < 2^32
  const uint32_t target = even < kAccTarget ? kAccTarget : even < kAccMost ? even : kAccMost;
  // one global add per block: an add per tile is 15 us of adds to one address
  const bool whole = total <= target && total != 0u;
  if (live && lane == 0) shared[bin] = !whole;
  __syncthreads();
  uint32_t at = 0;
  if (whole && lane == 0) at = atomicAdd(&wholes, 1u);
  __syncthreads();
  if (threadIdx.x == 0 && wholes != 0u) first_whole = atomicAdd(&queue->whole, wholes);
  __syncthreads();
  if (whole && lane == 0) items[cap - 1 - (int64_t)(first_whole + at)] = AccItem{bin, 0u, chunks, 0u};
  if (whole || !live) return;
  if (clear) clear_tile(clear, bin, l0, log2T, tb, lane, kWave);
  if (total == 0u) return;
  const uint32_t groups = total / target + 1u, per = total / groups + 1u;  // records
  uint32_t before = 0, start = 0, group = 0;  // records before the step, the open item's first chunk and group
  for (uint32_t cb = 0; cb < chunks; cb += kWave) {
    const uint32_t c = cb + lane;
    const uint2 q = c < chunks ? run[c] : make_uint2(0u, 0u);
    const uint32_t n = run_pairs(q) + run_singles(q), incl = (uint32_t)wave_incl_scan((int)n);
    const uint32_t mine = c < chunks ? (before + incl - n) / per : 0xffffffffu;  // < groups
    const uint32_t below = (uint32_t)__shfl_up((int)mine, 1, kWave);  // by every lane: an inactive one gives nothing
    const uint32_t prev = lane == 0 ? group : below;
    const bool opens = c < chunks && mine != prev;
    const uint64_t m = __ballot(opens);
    if (m != 0ull) {  // each closes the item before it
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&queue->split, (uint32_t)__popcll(m));
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
      const uint64_t lower = m & ((1ull << lane) - 1ull);
      const uint32_t from = lower ? cb + 63u - (uint32_t)__clzll((long long)lower) : start;
      if (opens) items[at + (uint32_t)__popcll(lower)] = AccItem{bin, from, c, 1u};
      start = cb + 63u - (uint32_t)__clzll((long long)m);
      group = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(start - cb));
    }
    before += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  }
  if (lane == 0) items[atomicAdd(&queue->split, 1u)] = AccItem{bin, start, chunks, 1u};
}

// The largest of the wave's values below 2^8.
__device__ __forceinline__ uint32_t wave_max8(uint32_t v) {
  uint32_t r = 0u;
  bool in = true;
#pragma unroll
  for (int b = 7; b >= 0; --b) {
    const bool one = in && ((v >> b) & 1u) != 0u;
    if (__any(one)) {
      r |= 1u << b;
      in = one;
    }
  }
  return r;
}

// The block's waves share a window of 64 pieces, a piece being up to 64
// consecutive records of a run; a batch is the pieces of up to kAccRuns runs
// (chunks).  Four waves scan the runs' numbers of pieces into LDS, then each
// lane of a wave looks up one piece of the window, and the wave reads its
// eight from those lanes.
// An item's windows are added one after the other without a barrier, all with
// the item's scale; its sums are converted and stored once.  The next item's
// first records and the runs of the batch after it are loaded before that, so
// their latency hides behind it.  A NaN or an infinity (only where the item
// says so) stays out of the sums and sets a bit of its entry.
// A workgroup takes items by place and then from a queue, the shared tiles'
// first, which are the longest.  Bound by the chain of an item (its runs, their places, its records, the LDS
// adds, the conversion), two workgroups per CU by LDS.
__global__ void __launch_bounds__(kAccBlock, 4) bin_accum_kernel(BinQueue *__restrict__ queue,
                                                                const AccItem *__restrict__ list, int64_t cap,
                                                                const uint2 *__restrict__ runs,
                                                                const char *__restrict__ rec, int64_t S,
                                                                const int64_t *__restrict__ S_dev, int64_t chunk_cap,
                                                                int l0, int nl, int log2T, int tb, int overwrite,
                                                                float *__restrict__ gtable) {
  extern __shared__ unsigned long long acc[];  // 2 E fixed-point sums: first features, second features
  __shared__ uint32_t special[3][kAccSums / 32];  // of each sum: an infinity, a negative one, a NaN came in
  __shared__ AccItem queued;  // the item after the next (bin kNoItem: none)
  __shared__ uint32_t trun[kAccRuns];  // the batch's runs (first record, count << 16)
  __shared__ int toff[kAccRuns];       // their first pieces, within the 64 runs of a wave
  __shared__ int ttot[kRunWaves];      // pieces of each 64 runs; whether they have single records
  __shared__ int tsing[kRunWaves];
  __shared__ uint32_t tex[kRunWaves];  // of the item: largest exponent field, kOdd
  constexpr uint32_t kOdd = 1u << 8;
  const int tpl_log2 = log2T - tb;
  const int n2 = 1 << tb;  // entries of a tile (2 sums each)
  const int n4 = n2 / 2;   // float4 (2 entries) per tile
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int64_t Sn = count_of(S, S_dev);
  const uint32_t chunks = (uint32_t)ceil_div(Sn, (int64_t)kSortChunk);
  const uint32_t nsplit = queue->split, nitems = nsplit + queue->whole;
  ulonglong2 *a2 = reinterpret_cast<ulonglong2 *>(acc);  // cleared while the counts are on their way
  for (int j = tid; j < n2; j += kAccBlock) a2[j] = make_ulonglong2(0ull, 0ull);
  for (int j = tid; j < kAccSums / 32; j += kAccBlock) special[0][j] = special[1][j] = special[2][j] = 0u;
  // a plan of these positions always passes the checks here and in item_at;
  // they keep a missing one (IA355_TABLE_REUSE_PLAN alone) inside the buffers
  if (blockIdx.x >= nitems || nitems < nsplit || nitems > cap) return;
  auto item_at = [&](uint32_t i) {
    AccItem I = i < nsplit ? list[i] : i < nitems ? list[cap - 1 - (int64_t)(i - nsplit)] : AccItem{kNoItem, 0u, 0u, 0u};
    if (i < nitems && (I.bin >= (uint32_t)nl << tpl_log2 || I.c0 > I.c1 || I.c1 > chunks)) I = AccItem{0u, 0u, 0u, 1u};
    return I;
  };
  // Items before `fixed` are taken by place, the last rounds' from a queue: an
  // add to one address takes 10 ns, and a workgroup waits for its turn, but the
  // items differ (36,503 samples, three rounds: 37 us, with two of them by
  // queue 41; 262,143, three long ones: 117, all by place 128; 16,384 short
  // ones 100, all by queue 118).
  const uint32_t rounds = nitems / gridDim.x, fixed = (rounds > 3u ? rounds - 1u : 2u) * gridDim.x;
  auto index_after = [&](uint32_t i) {
    return i + gridDim.x < fixed ? i + gridDim.x : fixed + atomicAdd(&queue->next, 1u);
  };
  auto uniform = [](const AccItem &I) {
    return AccItem{(uint32_t)__builtin_amdgcn_readfirstlane((int)I.bin),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)I.c0),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)I.c1),
                   (uint32_t)__builtin_amdgcn_readfirstlane((int)I.split)};
  };
  uint32_t taken = blockIdx.x;  // in thread 0: index of the item that was queued last
  if (tid == 0) queued = item_at(taken = index_after(taken));
  __syncthreads();
  // run of chunk cb + 64 wid + lane, in the first kRunWaves waves
  auto load_runs = [&](const AccItem &I, uint32_t cb) {
    const uint32_t c = cb + wid * kWave + lane;
    uint2 q = make_uint2(0u, 0u);
    if (wid < kRunWaves && c < I.c1) q = runs[(int64_t)I.bin * chunk_cap + c];
    return q;
  };
  AccItem I = uniform(item_at(blockIdx.x)), In = I;  // the item, that of the next batch
  AccItem item_n = uniform(queued);                  // the next item
  uint32_t cb = I.c0, cbn = 0;
  int kind = 0;  // 0: pair records, 1: single records
  uint2 ri = load_runs(I, cb), rin = make_uint2(0u, 0u);
  int total = 0, next = 0;  // pieces of the batch; the next window's first
  int sing = 0;             // the batch has single records as well
  uint4 raw[kAccPer];
  uint32_t in = 0;  // bit k: raw[k] holds a record
  auto begin = [&](bool first) {  // the tables of batch (cb, kind), the first of the item; a barrier follows
    if (wid < kRunWaves) {
      if (first) {
        uint32_t ex = run_exponent(ri);
        bool odd = run_odd(ri);
        for (uint32_t c = cb + kAccRuns + wid * kWave + lane; c < I.c1; c += kAccRuns) {
          const uint2 q = runs[(int64_t)I.bin * chunk_cap + c];
          ex = max(ex, run_exponent(q));
          odd |= run_odd(q);
        }
        ex = wave_max8(ex) | (__any(odd) ? kOdd : 0u);
        if (lane == 0) tex[wid] = ex;
      }
      const uint32_t count = kind ? run_singles(ri) : run_pairs(ri), first = kind ? ri.y & 0x3fffu : ri.x & 0x1fffu;
      const int n = (int)(count + kWave - 1) / kWave;
      const int incl = wave_incl_scan(n);
      trun[wid * kWave + lane] = first | count << 16;
      toff[wid * kWave + lane] = incl - n;
      const int sing = __any(run_singles(ri)) != 0;
      if (lane == kWave - 1) {
        ttot[wid] = incl;
        tsing[wid] = sing;
      }
    }
    next = 0;
  };
  auto fill = [&]() {  // this wave's pieces of the next window
    in = 0u;
    int base[kRunWaves];
    total = sing = 0;
#pragma unroll
    for (int h = 0; h < kRunWaves; ++h) {
      base[h] = total;
      total += __builtin_amdgcn_readfirstlane(ttot[h]);
      sing |= __builtin_amdgcn_readfirstlane(tsing[h]);
    }
    if (next < total) {
      // lane l: piece next + l
      int jl = next + lane, t0 = 0;
      const bool live = jl < total;
      int sub = 0;
#pragma unroll
      for (int h = 1; h < kRunWaves; ++h)
        if (jl >= base[h]) {
          t0 = h * kWave;
          sub = base[h];
        }
      jl -= sub;
      // the last run that starts at or before it (runs without records share
      // the next one's first piece and come before it)
      int c = t0;
#pragma unroll
      for (int st = kWave / 2; st > 0; st >>= 1)
        if (toff[c + st] <= jl) c += st;
      const uint32_t x = trun[c], i0 = (uint32_t)(jl - toff[c]) * kWave;
      const int left = live ? (int)(x >> 16) - (int)i0 : 0;
      int at = c * (kSortChunk * kSampleBytes);  // bytes from the batch's first chunk
      if (kind == 0) {
        at += 16 * (int)((x & 0xffffu) + i0);
      } else {  // a chunk's single records lie downwards from its end
        const int64_t ns = Sn - (int64_t)(cb + c) * kSortChunk;
        at += (int)(ns < kSortChunk ? ns : kSortChunk) * kSampleBytes - 12 * (int)((x & 0xffffu) + i0 + 1u);
      }
      const char *region0 = rec + ((int64_t)(I.bin >> tpl_log2) * S + (int64_t)cb * kSortChunk) * kSampleBytes;
      const int step = kind == 0 ? 16 : -12;
#pragma unroll
      for (int k = 0; k < kAccPer; ++k) {
        const int n = __builtin_amdgcn_readlane(left, k * kAccWaves + wid);
        const int o = __builtin_amdgcn_readlane(at, k * kAccWaves + wid);
        // lanes past the piece load the region's first bytes, which stay
        // unused, as do the last four of a single record's sixteen
        raw[k] = load16(region0 + (lane < n ? o + lane * step : 0));
        in |= lane < n ? 1u << k : 0u;
      }
    }
    next += kAccPer * kAccWaves;
  };
  auto next_batch = [&]() {  // the batch after (I, cb, kind 1), its runs on their way
    cbn = cb + kAccRuns;
    In = I;
    if (cbn >= I.c1) {
      In.c0 = In.c1 = cbn = 0;
      if (item_n.bin != kNoItem) {
        In = item_n;
        cbn = In.c0;
        if (tid == 0) queued = item_at(taken = index_after(taken));  // read after the next barrier
      }
    }
    rin = load_runs(In, cbn);
  };
  uint32_t how = 0;  // the item's largest exponent field, kOdd
  auto item_how = [&]() {
    uint32_t ex = 0, odd = 0;
#pragma unroll
    for (int h = 0; h < kRunWaves; ++h) {
      const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)tex[h]);
      ex = max(ex, t & 0xffu);
      odd |= t & kOdd;
    }
    return ex | odd;
  };
  begin(true);
  __syncthreads();
  how = item_how();
  fill();
  if (next >= total && !sing) next_batch();
  for (;;) {
    // |value| < 2^(exponent - 126): with 2^s, s = 173 - exponent, a value is
    // below 2^47 and a sum of the item's below 2^63
    const int sc = 173 - (int)(how & 0xffu);
    const double scale = __longlong_as_double((long long)(1023 + sc) << 52);
    const bool odd = (how & kOdd) != 0;
    auto add = [&](uint32_t i, float f) {
      if (odd && !isfinite(f))
        atomicOr(&special[isnan(f) ? 2 : f < 0.0f ? 1 : 0][i >> 5], 1u << (i & 31u));
      else
        atomicAdd(&acc[i], to_fixed(f, scale));
    };
#pragma unroll
    for (int k = 0; k < kAccPer; ++k) {
      if (!((in >> k) & 1u)) continue;
      const float4 v = values(raw[k], kind);
      const uint32_t e = kind ? raw[k].z : raw[k].w;
      const uint32_t e0 = e & (uint32_t)(n2 - 1), e1 = (e >> 16) & (uint32_t)(n2 - 1);
      add(e0, v.x);
      add(n2 + e0, v.y);
      if (kind) continue;
      add(e1, v.z);
      add(n2 + e1, v.w);
    }
    if (next < total) {
      fill();
    } else {
      // move on: the batch's single records, the next batch or item
      const AccItem I_now = I;
      bool last = false, stop = false;  // last window of the item; no item left
      __syncthreads();                  // the adds are complete, the tables and the queued item free to change
      if (kind == 0 && sing) {
        kind = 1;
      } else {
        last = cb + kAccRuns >= I.c1;
        stop = last && item_n.bin == kNoItem;
        if (last) item_n = uniform(queued);
        I = In;
        cb = cbn;
        ri = rin;
        kind = 0;
      }
      if (!stop) begin(last);
      __syncthreads();  // the tables are written
      if (!stop) {
        if (last) how = item_how();
        fill();
      }
      if (last) {
        const double inv = __longlong_as_double((long long)(1023 - sc) << 52);
        float4 *dst =
            reinterpret_cast<float4 *>(gtable + ((((int64_t)l0 << log2T) + ((int64_t)I_now.bin << tb)) << 1));
#pragma unroll
        for (int q = 0; q < kAccWr; ++q) {
          const int j = tid + q * kAccBlock;
          if (j >= n4) continue;
          const ulonglong2 f = a2[j], g = a2[n4 + j];
          a2[j] = make_ulonglong2(0ull, 0ull);
          a2[n4 + j] = make_ulonglong2(0ull, 0ull);
          float4 o = make_float4(from_fixed(f.x, inv), from_fixed(g.x, inv), from_fixed(f.y, inv), from_fixed(g.y, inv));
          if (odd) {
            auto mend = [&](uint32_t i, float &v) {
              const uint32_t w = i >> 5, b = 1u << (i & 31u);
              const bool pos = (special[0][w] & b) != 0, neg = (special[1][w] & b) != 0, nan = (special[2][w] & b) != 0;
              v = nan || (pos && neg) ? NAN : pos ? INFINITY : neg ? -INFINITY : v;
            };
            mend(2 * j, o.x);
            mend(n2 + 2 * j, o.y);
            mend(2 * j + 1, o.z);
            mend(n2 + 2 * j + 1, o.w);
          }
          if (I_now.split) {
            float *df = reinterpret_cast<float *>(dst + j);
            if (o.x != 0.0f) atomicAdd(df, o.x);
            if (o.y != 0.0f) atomicAdd(df + 1, o.y);
            if (o.z != 0.0f) atomicAdd(df + 2, o.z);
            if (o.w != 0.0f) atomicAdd(df + 3, o.w);
          } else {  // the only writer of this tile
            if (!overwrite) {
              const float4 p = dst[j];
              o.x += p.x;
              o.y += p.y;
              o.z += p.z;
              o.w += p.w;
            }
            store_once(dst + j, o);
          }
        }
        if (stop) return;
        if (odd) {
          __syncthreads();  // the bits are read
          for (int j = tid; j < kAccSums / 32; j += kAccBlock) special[0][j] = special[1][j] = special[2][j] = 0u;
        }
        __syncthreads();  // the sums are clear
      }
    }
    // once a batch, when its last window is on its way: an item taken earlier
    // would wait longer behind this one
    if (next >= total && (kind != 0 || !sing)) next_batch();
  }
}

}  // namespace

extern "C" int32_t ia355_hashgrid_encode(const float *xc, const int16_t *bone, int64_t S, const int64_t *S_dev,
                                         int64_t ld, const void *table, int32_t table_dtype, int32_t L, int32_t F,
                                         int32_t log2T, double base_res, double growth, const float *aabb, void *feat,
                                         int32_t feat_dtype, ia355_stream_t stream) {
  if (S < 0 || ld < S || L <= 0 || L > kMaxLevels || F != 2 || log2T < 1 || log2T > 30) return IA355_ERR_INVALID_ARG;
  if (!table || (S > 0 && (!xc || !feat))) return IA355_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(table) & 15) != 0 || log2T < 2) return IA355_ERR_INVALID_ARG;  // block gathers
  if (table_dtype != IA355_F32 && table_dtype != IA355_F16) return IA355_ERR_INVALID_ARG;
  if (feat_dtype != IA355_F32 && feat_dtype != IA355_BF16) return IA355_ERR_INVALID_ARG;
  Levels lv;
  Box box;
  if (make_levels(L, log2T, base_res, growth, &lv) || make_box(aabb, &box)) return IA355_ERR_INVALID_ARG;
  if (S == 0) return IA355_OK;
  const int per_xcd = (L + kXcd - 1) / kXcd;
  // two levels per lane where an XCD serves several levels
  const int lv_lane = per_xcd >= 2 ? 2 : 1;
  const int ngroup = (per_xcd + lv_lane - 1) / lv_lane;
  // two samples per lane as well for frame-sized calls (more gathers in
  // flight per lane; at training-step sizes the halved lane count costs more)
  const int sp_lane = lv_lane == 2 && S >= kTwoSampleMin ? 2 : 1;
  // chunk slots per (XCD, level group); with a device count the blocks loop
  // over what is left (blocks past the count exit at once)
  int64_t nslot = ceil_div(S, (int64_t)kFwdBlock * sp_lane);
  if (S_dev) {
    const int64_t quarter = table_dtype == IA355_F16 ? nslot / 4 : 0;
    const int64_t most = quarter < kDevSlots ? kDevSlots : quarter < kDevSlotsMost ? quarter : kDevSlotsMost;
    if (nslot > most) nslot = most;
  }
  const int64_t blocks = nslot * ngroup * kXcd;
  if (blocks > 0x7fffffffLL) return IA355_ERR_INVALID_ARG;
  hipStream_t s = as_stream(stream);
  const unsigned g = (unsigned)blocks;
  const EncodeArgs ea{xc, bone, S, S_dev, ld, table, L, log2T, lv, box, feat, ngroup};
  if (table_dtype == IA355_F32 && feat_dtype == IA355_F32)
    launch_encode<float, float>(ea, lv_lane, sp_lane, g, s);
  else if (table_dtype == IA355_F32)
    launch_encode<float, __hip_bfloat16>(ea, lv_lane, sp_lane, g, s);
  else if (feat_dtype == IA355_F32)
    launch_encode<__half, float>(ea, lv_lane, sp_lane, g, s);
  else
    launch_encode<__half, __hip_bfloat16>(ea, lv_lane, sp_lane, g, s);
  return launch_status();
}

extern "C" size_t ia355_hashgrid_encode_bwd_workspace_size(int64_t S, int32_t L) {
  if (S < 0 || L <= 0) return 0;
  return align256(sizeof(float) * 3 * (size_t)L * (size_t)(S > 0 ? S : 1));
}

extern "C" int32_t ia355_hashgrid_encode_bwd(const float *grad_feat, const float *xc, const int16_t *bone, int64_t S,
                                             const int64_t *S_dev, int64_t ld, const void *table, int32_t table_dtype,
                                             int32_t L, int32_t F, int32_t log2T, double base_res, double growth,
                                             const float *aabb, float *grad_table, float *grad_xc, uint32_t flags,
                                             void *ws, size_t ws_bytes, ia355_stream_t stream) {
  if (S < 0 || ld < S || L <= 0 || L > 16 || F != 2 || log2T < 1 || log2T > 30) return IA355_ERR_INVALID_ARG;
  if (S > 0 && (!grad_feat || !xc)) return IA355_ERR_INVALID_ARG;
  if (grad_xc && !table) return IA355_ERR_INVALID_ARG;
  if (grad_xc && ((reinterpret_cast<uintptr_t>(table) & 15) != 0 || log2T < 2)) return IA355_ERR_INVALID_ARG;
  if (grad_xc && S > 0 && (!ws || ws_bytes < ia355_hashgrid_encode_bwd_workspace_size(S, L)))
    return IA355_ERR_WORKSPACE;
  if (table_dtype != IA355_F32 && table_dtype != IA355_F16) return IA355_ERR_INVALID_ARG;
  const uint32_t known = IA355_OVERWRITE | IA355_TABLE_COARSE | IA355_TABLE_FINE;
  if (flags & ~known) return IA355_ERR_INVALID_ARG;
  Levels lv;
  Box box;
  if (make_levels(L, log2T, base_res, growth, &lv) || make_box(aabb, &box)) return IA355_ERR_INVALID_ARG;
  hipStream_t s = as_stream(stream);
  const bool dev = S_dev != nullptr;
  const int overwrite = (flags & IA355_OVERWRITE) != 0;
  // Run aggregation pays while a cell spans several ray steps (coarse dense
  // levels, which come first as the resolution grows with the level); finer
  // levels use the 16-lanes-per-item mapping.  The two groups touch disjoint
  // slices of the table, so a caller may run them on two streams.
  int ndense = 0;
  while (ndense < L && lv.dense[ndense] && lv.res[ndense] <= kAggMaxRes) ++ndense;
  const bool coarse = !(flags & IA355_TABLE_FINE) || (flags & IA355_TABLE_COARSE);
  const bool fine = !(flags & IA355_TABLE_COARSE) || (flags & IA355_TABLE_FINE);
  const int l0 = coarse ? 0 : ndense, l1 = fine ? L : ndense;
  const size_t level_floats = 2 * ((size_t)1 << log2T);
  if (grad_table && overwrite && l1 > l0) {
    const int32_t st = ia355_zero(grad_table + level_floats * l0, sizeof(float) * level_floats * (l1 - l0), stream);
    if (st != IA355_OK) return st;
  }
  if (grad_table && S > 0) {
    // The atomics do not return values, so a few waves per CU keep the
    // memory-side atomic units busy; bounded grids (grid-stride) leave CUs
    // to kernels on other streams (the position gradient and the IFT run
    // beside the table gradient).
    if (coarse && ndense > 0)
      table_grad_dense_kernel<<<stride_grid(ceil_div(S, kDgBlock) * ndense, true, kTgDenseMaxGrid), kDgBlock, 0, s>>>(
          grad_feat, xc, bone, S, S_dev, ld, ndense, log2T, lv, box, grad_table);
    if (fine && ndense < L)
      table_grad_kernel<<<stride_grid(ceil_div((int64_t)(L - ndense) * S * 16, kTgBlock), true, kTgMaxGrid), kTgBlock,
                          0, s>>>(grad_feat, xc, bone, S, S_dev, ld, ndense, L, log2T, lv, box, grad_table);
  }
  if (grad_xc && S > 0) {
    float *part = (float *)ws;
    const int per_xcd = (L + kXcd - 1) / kXcd;
    const int lv_lane = per_xcd >= 2 ? 2 : 1;
    const int ngroup = (per_xcd + lv_lane - 1) / lv_lane;
    int64_t nslot = ceil_div(S, kBwdBlock);
    if (dev && nslot > 1024) nslot = 1024;
    const int64_t blocks = nslot * ngroup * kXcd;
    if (blocks > 0x7fffffffLL) return IA355_ERR_INVALID_ARG;
    if (table_dtype == IA355_F32)
      launch_xgrad<float>(lv_lane, (unsigned)blocks, s, grad_feat, xc, bone, S, S_dev, ld, table, L, log2T, lv, box,
                          part, ngroup);
    else
      launch_xgrad<__half>(lv_lane, (unsigned)blocks, s, grad_feat, xc, bone, S, S_dev, ld, table, L, log2T, lv, box,
                           part, ngroup);
    xgrad_sum_kernel<<<stride_grid(ceil_div(S, kBwdBlock), dev, 1024), kBwdBlock, 0, s>>>(part, S, S_dev, L, ld,
                                                                                           grad_xc);
  }
  return launch_status();
}

extern "C" size_t ia355_hashgrid_table_grad_workspace_size(int64_t S, int32_t L, int32_t log2T) {
  BinGeom g;
  if (L <= 0 || L > 16 || !bin_geom(L, S, log2T, &g)) return 0;
  return bin_ws(L, S, g, nullptr).bytes;
}

extern "C" int32_t ia355_hashgrid_table_grad(const float *grad_feat, const float *xc, const int16_t *bone, int64_t S,
                                             const int64_t *S_dev, int64_t ld, int32_t L, int32_t F, int32_t log2T,
                                             double base_res, double growth, const float *aabb, float *grad_table,
                                             uint32_t flags, void *ws, size_t ws_bytes, ia355_stream_t stream) {
  const uint32_t known =
      IA355_OVERWRITE | IA355_TABLE_COARSE | IA355_TABLE_FINE | IA355_TABLE_PLAN | IA355_TABLE_REUSE_PLAN;
  if (flags & ~known) return IA355_ERR_INVALID_ARG;
  const bool plan_only = (flags & IA355_TABLE_PLAN) != 0, reuse = (flags & IA355_TABLE_REUSE_PLAN) != 0;
  if (plan_only && reuse) return IA355_ERR_INVALID_ARG;
  if (S < 0 || ld < S || L <= 0 || L > 16 || F != 2 || log2T < 2 || log2T > 30) return IA355_ERR_INVALID_ARG;
  if (S > 0 && !xc) return IA355_ERR_INVALID_ARG;
  if (!plan_only && (!grad_table || (S > 0 && !grad_feat))) return IA355_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(grad_table) & 15) != 0) return IA355_ERR_INVALID_ARG;  // float4 tile stores
  Levels lv;
  Box box;
  if (make_levels(L, log2T, base_res, growth, &lv) || make_box(aabb, &box)) return IA355_ERR_INVALID_ARG;
  BinGeom full;
  if (!bin_geom(L, S, log2T, &full)) return IA355_ERR_INVALID_ARG;
  if (!ws || ws_bytes < bin_ws(L, S, full, nullptr).bytes) return IA355_ERR_WORKSPACE;
  int ndense = 0;
  while (ndense < L && lv.dense[ndense] && lv.res[ndense] <= kAggMaxRes) ++ndense;
  const bool coarse = !(flags & IA355_TABLE_FINE) || (flags & IA355_TABLE_COARSE);
  const bool fine = !(flags & IA355_TABLE_COARSE) || (flags & IA355_TABLE_FINE);
  const int l0 = coarse ? 0 : ndense, l1 = fine ? L : ndense;
  if (l1 <= l0) return IA355_OK;
  const int overwrite = (flags & IA355_OVERWRITE) != 0;
  hipStream_t s = as_stream(stream);
  if (S == 0) {
    if (plan_only || !overwrite) return IA355_OK;
    const size_t level_floats = 2 * ((size_t)1 << log2T);
    return ia355_zero(grad_table + level_floats * l0, sizeof(float) * level_floats * (l1 - l0), stream);
  }
  const int nl = l1 - l0;
  BinGeom g;
  bin_geom(nl, S, log2T, &g);  // fewer levels than `full`: fits its workspace
  const BinWs w = bin_ws(nl, S, g, ws);
  const size_t cnt_lds = sizeof(uint2) * ((size_t)1 << g.tpl_log2), most_lds = sizeof(uint2) * kMaxBins;  // 128 KB
  // the blocks loop over the chunks; with a device count the grid is bounded
  int64_t per_level = g.chunks < 4096 ? g.chunks : 4096;
  if (S_dev && per_level > 64) per_level = 64;
  auto *sort = plan_only ? bin_sort_kernel<kBinPlan> : reuse ? bin_sort_kernel<kBinRest> : bin_sort_kernel<kBinAll>;
  if (cnt_lds > 48 * 1024 &&
      hipFuncSetAttribute((const void *)sort, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most_lds) != hipSuccess)
    return IA355_ERR_HIP;
  sort<<<(unsigned)(nl * per_level), kSortBlock, cnt_lds, s>>>(grad_feat, xc, bone, S, S_dev, ld, l0, nl, log2T, g.tb,
                                                               lv, box, g.chunks, w.queue, w.runs, w.rec, w.shared,
                                                               overwrite ? grad_table : nullptr);
  if (!reuse)
    bin_plan_kernel<<<(unsigned)ceil_div((int64_t)nl << g.tpl_log2, kPlanBlock / kWave), kPlanBlock, 0, s>>>(
        w.runs, S, S_dev, g.chunks, l0, nl, log2T, g.tb, w.cap, w.queue, w.items, w.shared,
        overwrite && !plan_only ? grad_table : nullptr);
  if (!plan_only)
    bin_accum_kernel<<<kAccMaxGrid, kAccBlock, sizeof(unsigned long long) * 2 * ((size_t)1 << g.tb), s>>>(
        w.queue, w.items, w.cap, w.runs, w.rec, S, S_dev, g.chunks, l0, nl, log2T, g.tb, overwrite, grad_table);
  return launch_status();
}
