// Per-sample arithmetic of the root finding (Sec. 3.1, Eq. 5-7), shared by
// the deform kernels and the persistent batch renderer so that both compute
// the same floats: the blended transform grid A_v = sum_i W[v][i] B_i, the
// residual g(x) = sum_c tri_c (A_c x_h) - x' and its Jacobian on that grid,
// one Broyden solve and the multi-init search (internal).
#pragma once
#include "common.h"
#include "geometry.h"

namespace ia355 {
namespace dfm {

constexpr int kMaxBones = 64;

struct Grid {
  int D[3];       // Dx, Dy, Dz
  float lo[3];    // box low corner
  float scale[3]; // (D - 1) / (hi - lo)
  uint32_t dc[8]; // byte offset of corner k's transform (k = cx + 2 cy + 4 cz) from its cell's base vertex
};

struct Box {
  float lo[3], hi[3];
};

// A_v of one vertex from its skinning row w [nb] and the bone transforms
// sB [nb][12]: the weighted sum over bones in bone order.
__device__ __forceinline__ void blend_vertex(const float *w, const float *sB, int nb, float *Av) {
  float acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0f;
  for (int b = 0; b < nb; ++b) {
    const float wb = w[b];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] += wb * sB[12 * b + k];
  }
  float4 *out = reinterpret_cast<float4 *>(Av);
  out[0] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  out[1] = make_float4(acc[4], acc[5], acc[6], acc[7]);
  out[2] = make_float4(acc[8], acc[9], acc[10], acc[11]);
}

// Vertices blk * kBlendBlock ... of the blended grid A, one thread per
// vertex (a block of kBlendBlock threads).  The block's nb-float skinning
// rows are contiguous in W, so the block first copies them into LDS with
// coalesced 16-byte loads (a lane walking its own row would touch a
// different cache line per lane and weight), then each thread blends its row
// with the bone transforms.  sB [kMaxBones * 12] and
// sW [kBlendBlock * kBlendMaxBones] are the block's LDS.
constexpr int kBlendBlock = 256;
constexpr int kBlendMaxBones = 32;  // LDS rows: 256 x 32 floats = 32 KB
__device__ __forceinline__ void blend_block(const float *__restrict__ W, const float *__restrict__ B, int nb,
                                            int64_t nvert, float *__restrict__ A, int64_t blk, float *sB, float *sW) {
  for (int i = threadIdx.x; i < nb * 12; i += blockDim.x) sB[i] = B[i];
  const int64_t v0 = blk * kBlendBlock;
  const int64_t nv = nvert - v0 < kBlendBlock ? nvert - v0 : kBlendBlock;
  const bool staged = nb <= kBlendMaxBones;
  if (staged) {
    // the block's rows: nv * nb floats starting at W + v0 * nb
    const float *src = W + v0 * nb;
    const int64_t n = nv * nb;
    const int64_t head = (int64_t)((4 - (((uintptr_t)src >> 2) & 3)) & 3);  // floats before 16-byte alignment
    const int64_t h = head < n ? head : n;
    for (int64_t i = threadIdx.x; i < h; i += blockDim.x) sW[i] = src[i];
    const int64_t n4 = (n - h) >> 2;
    const float4 *src4 = reinterpret_cast<const float4 *>(src + h);
    for (int64_t i = threadIdx.x; i < n4; i += blockDim.x) {
      const float4 q = src4[i];
      sW[h + 4 * i] = q.x;
      sW[h + 4 * i + 1] = q.y;
      sW[h + 4 * i + 2] = q.z;
      sW[h + 4 * i + 3] = q.w;
    }
    for (int64_t i = h + 4 * n4 + threadIdx.x; i < n; i += blockDim.x) sW[i] = src[i];
  }
  __syncthreads();
  const int64_t v = v0 + threadIdx.x;
  if (threadIdx.x < nv) blend_vertex(staged ? sW + (int64_t)threadIdx.x * nb : W + v * nb, sB, nb, A + 12 * v);
}

// Cell lookup with align-corners vertices and clamping to the box: base
// vertex, fractional position and d(p)/dx (zero along a clamped axis).
struct Cell {
  int i0[3];
  float f[3];
  float dp[3];
};

__device__ __forceinline__ Cell locate(const Grid &g, const float x[3]) {
#pragma clang fp contract(off)
  Cell c;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    float p = (x[a] - g.lo[a]) * g.scale[a];
    float s = g.scale[a];
    const float pmax = (float)(g.D[a] - 1);
    if (!(p >= 0.0f)) { p = 0.0f; s = 0.0f; }  // also catches NaN
    if (p > pmax) { p = pmax; s = 0.0f; }
    int i = (int)floorf(p);
    i = i > g.D[a] - 2 ? g.D[a] - 2 : i;
    i = i < 0 ? 0 : i;
    c.i0[a] = i;
    c.f[a] = p - (float)i;
    c.dp[a] = s;
  }
  return c;
}

// Base vertex of a cell.  The blended grid holds fewer than 2^32 / 48
// vertices (checked on the host), so vertex and byte offsets are 32-bit and
// every corner load is a uniform base plus one 32-bit lane offset.
// (byte offset of the base vertex's 12 floats)
__device__ __forceinline__ uint32_t cell_base(const Grid &g, const Cell &c) {
  return (((uint32_t)c.i0[2] * (uint32_t)g.D[1] + (uint32_t)c.i0[1]) * (uint32_t)g.D[0] + (uint32_t)c.i0[0]) * 48u;
}

// Sources of a cell's eight corner transforms for the residuals below: start()
// and at() name the cell (byte offset of its base vertex), corner() gives the
// three rows of corner k.  at() changes the cell of the lanes with `need`; it is
// called by the whole wave.  Every source gives the same floats.
//  * HeldCorners keeps the last cell's 96 floats in registers and gathers
//    only when the cell changes.  The time went to the texture path (24
//    gathers of 16 bytes per residual), and Broyden's steps shrink so fast
//    that only the start, the first step and a fifth of the second steps reach
//    a new cell of a 64 x 64 x 32 grid.  It costs 60 to 70 registers (guided
//    solve 91 -> 166, three waves per SIMD; multi-init solve 121 -> 174, two)
//    and pays all the same: against gathering, guided solve of 875,600 samples
//    133 -> 76 us, multi-init solve of 36,503 83 -> 72, of a 64^3 lattice 477
//    -> 398.  The root lists, the guided solve's fallback, and the small calls
//    of the multi-init and of the guided solve use it.
//  * SharedCorners adds to it: the cells that a wave's lanes lack are loaded
//    once each into LDS (24 lanes load a cell's 384 bytes directly) and read
//    from there into the lanes' registers.  After kCellSlots distinct cells
//    the lanes left gather their own.  The guided solve uses it beyond 65,536
//    samples; a wave's 64 lie in few cells: 875,600 samples 75 -> 43 us, of a
//    frame 78 -> 65; in random order a whole guided pass takes 124 us as it
//    did before (24 slots: 132).
//  * SharedLater, which the multi-init solve uses but for few samples of few
//    bones (168 registers, three waves), gathers the start cells, which differ
//    in nearly every lane, and shares the later ones: 14 cells a wave at the
//    first step and 6 at the second (24 slots in place of 12: 36,503 samples
//    67 us against 64, eight: 65).
//  * GatherCorners reads them from the blended grid each time: the persistent
//    renderer, whose other stages leave no registers to hold a cell.
struct GatherCorners {
  const float *A;
  const uint32_t *dc;
  uint32_t base;
  __device__ __forceinline__ GatherCorners(const float *A_, const Grid &g) : A(A_), dc(g.dc), base(0) {}
  __device__ __forceinline__ void start(uint32_t b) { base = b; }
  __device__ __forceinline__ void at(uint32_t b, bool need) { base = need ? b : base; }
  __device__ __forceinline__ void corner(int k, float4 r[3]) const {
    const float4 *p = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(A) + (base + dc[k]));
    r[0] = p[0];
    r[1] = p[1];
    r[2] = p[2];
  }
};

struct HeldCorners {
  const float *A;
  const uint32_t *dc;
  uint32_t base;
  float4 v[8][3];
  __device__ __forceinline__ HeldCorners(const float *A_, const Grid &g) : A(A_), dc(g.dc) {}
  __device__ __forceinline__ void start(uint32_t b) {
    base = b;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float4 *p = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(A) + (b + dc[k]));
      v[k][0] = p[0];
      v[k][1] = p[1];
      v[k][2] = p[2];
    }
  }
  __device__ __forceinline__ void at(uint32_t b, bool need) {
    if (need && b != base) start(b);
  }
  __device__ __forceinline__ void corner(int k, float4 r[3]) const {
    r[0] = v[k][0];
    r[1] = v[k][1];
    r[2] = v[k][2];
  }
};

constexpr int kCellSlots = 12;   // distinct cells of a wave loaded through LDS at a time
constexpr int kCellBytes = 400;  // 8 x 48, and 16 to spread the slots over the banks
struct CellLds {
  __attribute__((aligned(16))) unsigned char slot[kCellSlots][kCellBytes];
};

struct SharedCorners : HeldCorners {
  CellLds &lds;   // of this wave
  uint32_t part;  // byte offset from a cell's base vertex of the 16 bytes that this lane loads (of 24 lanes)
  __device__ __forceinline__ SharedCorners(const float *A_, const Grid &g, CellLds &l) : HeldCorners(A_, g), lds(l) {
    const int ln = threadIdx.x & (kWave - 1), k = ln < 24 ? ln / 3 : 0;
    part = 16u * (uint32_t)(ln % 3);
#pragma unroll
    for (int c = 1; c < 8; ++c) part += k == c ? g.dc[c] : 0u;
  }
  __device__ __forceinline__ void start(uint32_t b) {
    base = 0xffffffffu;
    at(b, true);
  }
  __device__ __forceinline__ void at(uint32_t b, bool need) {
    const int ln = threadIdx.x & (kWave - 1);
    uint64_t rem = __builtin_amdgcn_ballot_w64(need && b != base);
    if (rem == 0ull) return;
    int slot = -1;
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the slots' last readers are done
    int s = 0;
    do {
      const uint32_t sb = (uint32_t)__builtin_amdgcn_readlane((int)b, __builtin_ctzll(rem));
      const bool same = b == sb;  // a lane without need may join: its copy stays that of its cell
      slot = same ? s : slot;
      rem &= ~__builtin_amdgcn_ballot_w64(same);
      if (ln < 24)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void *)(reinterpret_cast<const char *>(A) + (sb + part)),
            (__attribute__((address_space(3))) void *)(lds.slot[s]), 16, 0, 0);
    } while (++s < kCellSlots && rem != 0ull);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    asm volatile("" ::: "memory");
    if (slot >= 0) {
      base = b;
      const float4 *q = reinterpret_cast<const float4 *>(lds.slot[slot]);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i) v[k][i] = q[3 * k + i];
    }
    if (rem != 0ull) HeldCorners::at(b, need);
  }
};

struct SharedLater : SharedCorners {
  using SharedCorners::SharedCorners;
  __device__ __forceinline__ void start(uint32_t b) { HeldCorners::start(b); }
};

// Trilinear weights of the eight corners (k = cx + 2 cy + 4 cz).
__device__ __forceinline__ void tri_weights(const float f[3], float t[8]) {
  const float gx = 1.0f - f[0], gy = 1.0f - f[1], gz = 1.0f - f[2];
  const float a00 = gy * gz, a10 = f[1] * gz, a01 = gy * f[2], a11 = f[1] * f[2];
  t[0] = gx * a00;
  t[1] = f[0] * a00;
  t[2] = gx * a10;
  t[3] = f[0] * a10;
  t[4] = gx * a01;
  t[5] = f[0] * a01;
  t[6] = gx * a11;
  t[7] = f[0] * a11;
}

__device__ __forceinline__ void fma4(float t, const float4 &r, float4 &m) {
  m.x = fmaf(t, r.x, m.x);
  m.y = fmaf(t, r.y, m.y);
  m.z = fmaf(t, r.z, m.z);
  m.w = fmaf(t, r.w, m.w);
}

// The residual, its Jacobian and the Broyden iteration fix every rounding
// (fmaf and dot3, no contraction): the staged kernels and the persistent
// renderer hold the corner values differently and must agree bit for bit.

// g = (sum_c tri_c A_c) x_h - x': the 12 blended channels are interpolated
// first, then applied to x_h once.
template <class Corners>
__device__ __forceinline__ void residual(const Corners &cs, const Cell &c, const float x[3], const float xp[3],
                                         float g[3]) {
#pragma clang fp contract(off)
  float t[8];
  tri_weights(c.f, t);
  float4 m0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), m1 = m0, m2 = m0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float4 r[3];
    cs.corner(k, r);
    fma4(t[k], r[0], m0);
    fma4(t[k], r[1], m1);
    fma4(t[k], r[2], m2);
  }
  g[0] = (dot3(m0.x, x[0], m0.y, x[1], m0.z, x[2]) + m0.w) - xp[0];
  g[1] = (dot3(m1.x, x[0], m1.y, x[1], m1.z, x[2]) + m1.w) - xp[1];
  g[2] = (dot3(m2.x, x[0], m2.y, x[1], m2.z, x[2]) + m2.w) - xp[2];
}

// Derivatives of a trilinear interpolant along its cell axes, from the
// eight corner values v[c] (c = cx + 2 cy + 4 cz) and the fractions f:
// differences of neighbouring corners are taken first, so the result does
// not cancel when the corner values are close (they are smooth fields).
__device__ __forceinline__ void tri_grad(const float v[8], const float f[3], float d[3]) {
#pragma clang fp contract(off)
  const float gx = 1.0f - f[0], gy = 1.0f - f[1], gz = 1.0f - f[2];
  d[0] = fmaf(f[1] * f[2], v[7] - v[6], dot3(gy * gz, v[1] - v[0], f[1] * gz, v[3] - v[2], gy * f[2], v[5] - v[4]));
  d[1] = fmaf(f[0] * f[2], v[7] - v[5], dot3(gx * gz, v[2] - v[0], f[0] * gz, v[3] - v[1], gx * f[2], v[6] - v[4]));
  d[2] = fmaf(f[0] * f[1], v[7] - v[3], dot3(gx * gy, v[4] - v[0], f[0] * gy, v[5] - v[1], gx * f[1], v[6] - v[2]));
}

__device__ __forceinline__ float tri_weight(const float f[3], int k) {
  return ((k & 1) ? f[0] : 1.0f - f[0]) * ((k & 2) ? f[1] : 1.0f - f[1]) * ((k & 4) ? f[2] : 1.0f - f[2]);
}

// Residual and Jacobian: with y_c = A_c x_h, g = sum_c tri_c y_c - x' and
// J = sum_c tri_c M_c + (d/dx of the interpolant of y_c at fixed x_h).
template <class Corners>
__device__ __forceinline__ void residual_jac(Corners &cs, const Grid &gr, const float x[3], const float xp[3], float g[3],
                                             float J[3][3]) {
#pragma clang fp contract(off)
  const Cell c = locate(gr, x);
  cs.start(cell_base(gr, c));
  float y[3][8];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) J[i][j] = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float4 r[3];
    cs.corner(k, r);
    const float t = tri_weight(c.f, k);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      y[i][k] = dot3(r[i].x, x[0], r[i].y, x[1], r[i].z, x[2]) + r[i].w;
      J[i][0] = fmaf(t, r[i].x, J[i][0]);
      J[i][1] = fmaf(t, r[i].y, J[i][1]);
      J[i][2] = fmaf(t, r[i].z, J[i][2]);
    }
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float d[3];
    tri_grad(y[i], c.f, d);
    g[i] = -xp[i];
#pragma unroll
    for (int k = 0; k < 8; ++k) g[i] = fmaf(tri_weight(c.f, k), y[i][k], g[i]);
#pragma unroll
    for (int j = 0; j < 3; ++j) J[i][j] = fmaf(c.dp[j], d[j], J[i][j]);
  }
}

__device__ __forceinline__ float norm3(const float v[3]) { return sqrtf(dot3(v[0], v[0], v[1], v[1], v[2], v[2])); }

constexpr int kSolveBlock = 256;
// kGroup lanes share one posed sample; lane j runs inits j, j + kGroup, ...
// (3 of the 24 bones each), then the group selects the lowest residual by
// shuffles.  Many more threads than samples keep the CUs busy at the
// training-step sample counts (tens of thousands).
constexpr int kGroup = 8;

struct InitResult {
  float x[3];
  float r;
  bool ok;
  int steps;
};

// One Broyden solve from the start point x (H0 = J(x)^{-1}).
template <class Corners>
__device__ __forceinline__ InitResult broyden_from(Corners &cs, const Grid &gr, float x[3], bool start_ok,
                                                  const float xp[3], int max_iter, float tol_stop) {
#pragma clang fp contract(off)
  InitResult res;
  const bool bone_ok = start_ok;
  float g[3], J[3][3], H[3][3];
  residual_jac(cs, gr, x, xp, g, J);
  const float detJ = inv3(J, H);
  bool ok = bone_ok && fabsf(detJ) >= 1e-12f;
  int steps = 0;
  const float tol2 = tol_stop * tol_stop;
  // the lanes iterate together (at() may need them all); run: not done yet
  bool run = ok;
  for (int k = 0; k < max_iter; ++k) {
    run = run && !(dot3(g[0], g[0], g[1], g[1], g[2], g[2]) < tol2);
    if (!__any(run)) break;
    float dx[3], xn[3];
    Cell c;
    if (run) {
#pragma unroll
      for (int a = 0; a < 3; ++a) dx[a] = -dot3(H[a][0], g[0], H[a][1], g[1], H[a][2], g[2]);
#pragma unroll
      for (int a = 0; a < 3; ++a) xn[a] = x[a] + dx[a];
      c = locate(gr, xn);
    }
    cs.at(run ? cell_base(gr, c) : 0u, run);
    if (run) {
      float gn[3], dg[3], Hdg[3], dxH[3];
      residual(cs, c, xn, xp, gn);
#pragma unroll
      for (int a = 0; a < 3; ++a) dg[a] = gn[a] - g[a];
#pragma unroll
      for (int a = 0; a < 3; ++a) Hdg[a] = dot3(H[a][0], dg[0], H[a][1], dg[1], H[a][2], dg[2]);
#pragma unroll
      for (int b = 0; b < 3; ++b) dxH[b] = dot3(dx[1], H[1][b], dx[0], H[0][b], dx[2], H[2][b]);
      const float den = dot3(dx[1], Hdg[1], dx[0], Hdg[0], dx[2], Hdg[2]);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        x[a] = xn[a];
        g[a] = gn[a];
      }
      ++steps;
      if (fabsf(den) < 1e-30f) {
        ok = run = false;
      } else {
        const float iden = __builtin_amdgcn_rcpf(den);  // 1 ulp: H is an approximation of J^-1 anyway
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int b = 0; b < 3; ++b) H[a][b] = fmaf((dx[a] - Hdg[a]) * dxH[b], iden, H[a][b]);
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) res.x[a] = x[a];
  res.r = norm3(g);
  res.ok = ok;
  res.steps = steps;
  return res;
}

// One Broyden solve from bone init i: x0 = B_i^{-1} x'.
template <class Corners>
__device__ __forceinline__ InitResult broyden(Corners &cs, const Grid &gr, const float *Bi, bool bone_ok,
                                             const float xp[3], int max_iter, float tol_stop) {
  float x[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) x[a] = dot3(Bi[4 * a], xp[0], Bi[4 * a + 1], xp[1], Bi[4 * a + 2], xp[2]) + Bi[4 * a + 3];
  return broyden_from(cs, gr, x, bone_ok, xp, max_iter, tol_stop);
}

__device__ __forceinline__ bool in_hbox(const float x[3], const Box &b) {
  return x[0] >= b.lo[0] && x[0] <= b.hi[0] && x[1] >= b.lo[1] && x[1] <= b.hi[1] && x[2] >= b.lo[2] &&
         x[2] <= b.hi[2];
}

// Multi-init solve of one sample by a group of `lanes` lanes (a power of two,
// uniform; j = lane in group): lowest valid residual, ties to the lowest bone.
// Every lane of the group returns the group's result; steps are summed over the
// inits.
struct Choice {
  float x[3], r, x0[3];
  int bone, steps;
};

// Where a lane keeps its best root and init 0's last iterate between inits:
// registers, or LDS (seldom touched; the multi-init solve has none to spare).
struct RegKeep {
  float v[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  __device__ __forceinline__ void set(int k, float x) { v[k] = x; }
  __device__ __forceinline__ float get(int k) const { return v[k]; }
};
struct LdsKeep {
  float *p;  // [6][kSolveBlock], at this thread's column
  __device__ __forceinline__ explicit LdsKeep(float *base) : p(base + threadIdx.x) {
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k * kSolveBlock] = 0.0f;
  }
  __device__ __forceinline__ void set(int k, float x) { p[k * kSolveBlock] = x; }
  __device__ __forceinline__ float get(int k) const { return p[k * kSolveBlock]; }
};

template <class Corners, class Keep>
__device__ __forceinline__ Choice multi_init(Corners &cs, Keep kept, const Grid &gr, const float *sBinv,
                                             const int *sBok, int nb, const float xp[3], bool act, int lanes, int j,
                                             Box hbox, int max_iter, float tol_stop, float tol_valid) {
  float best_r = INFINITY;
  int best = 0x7fffffff, steps = 0;
  // (the same number of inits for every lane: at() may need them all)
  for (int i0 = 0; i0 < nb; i0 += lanes) {
    const bool mine = act && i0 + j < nb;
    const int i = mine ? i0 + j : 0;
    const InitResult q = broyden(cs, gr, sBinv + 12 * i, mine && sBok[i], xp, max_iter, tol_stop);
    if (!mine) continue;
    steps += q.steps;
    if (i == 0)
#pragma unroll
      for (int a = 0; a < 3; ++a) kept.set(3 + a, q.x[a]);
    if (q.ok && q.r < tol_valid && in_hbox(q.x, hbox) && q.r < best_r) {
      best_r = q.r;
      best = i;
#pragma unroll
      for (int a = 0; a < 3; ++a) kept.set(a, q.x[a]);
    }
  }
  float best_x[3], x0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    best_x[a] = kept.get(a);
    x0[a] = kept.get(3 + a);
  }
  for (int o = lanes / 2; o > 0; o >>= 1) {
    const float r2 = __shfl_xor(best_r, o, kWave);
    const int b2 = __shfl_xor(best, o, kWave);
    const float x20 = __shfl_xor(best_x[0], o, kWave);
    const float x21 = __shfl_xor(best_x[1], o, kWave);
    const float x22 = __shfl_xor(best_x[2], o, kWave);
    steps += __shfl_xor(steps, o, kWave);
    if (r2 < best_r || (r2 == best_r && b2 < best)) {
      best_r = r2;
      best = b2;
      best_x[0] = x20;
      best_x[1] = x21;
      best_x[2] = x22;
    }
  }
  Choice c;
  const bool valid = best != 0x7fffffff;
  // the group's first lane ran init 0: its final iterate stands for invalid samples
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c.x[a] = best_x[a];
    c.x0[a] = x0[a];
  }
  c.r = valid ? best_r : INFINITY;
  c.bone = valid ? best : -1;
  c.steps = steps;
  return c;
}

__device__ __forceinline__ void write_choice(const Choice &c, int64_t n, int64_t ld, int extra_steps, float *xc_soa,
                                             int16_t *bone_out, float *resid_out, int16_t *steps_out) {
  const bool valid = c.bone >= 0;
  xc_soa[n] = valid ? c.x[0] : c.x0[0];
  xc_soa[ld + n] = valid ? c.x[1] : c.x0[1];
  xc_soa[2 * ld + n] = valid ? c.x[2] : c.x0[2];
  bone_out[n] = (int16_t)c.bone;
  if (resid_out) resid_out[n] = c.r;
  if (steps_out) steps_out[n] = (int16_t)(c.steps + extra_steps);
}

inline Grid make_grid(int Dx, int Dy, int Dz, const float *aabb) {
  Grid g;
  g.D[0] = Dx;
  g.D[1] = Dy;
  g.D[2] = Dz;
  for (int a = 0; a < 3; ++a) {
    g.lo[a] = aabb[a];
    g.scale[a] = (float)(g.D[a] - 1) / (aabb[3 + a] - aabb[a]);
  }
  const uint32_t sx = 1, sy = (uint32_t)Dx, sz = (uint32_t)Dx * (uint32_t)Dy;
  for (int k = 0; k < 8; ++k) g.dc[k] = 48u * (((k & 1) ? sx : 0) + ((k & 2) ? sy : 0) + ((k & 4) ? sz : 0));
  return g;
}

inline bool grid_ok(int Dx, int Dy, int Dz, const float *aabb) {
  if (Dx < 2 || Dy < 2 || Dz < 2 || !aabb) return false;
  if ((int64_t)Dx * Dy * Dz * 48 >= ((int64_t)1 << 32)) return false;  // 32-bit byte offsets into the blended grid
  for (int a = 0; a < 3; ++a)
    if (!(aabb[3 + a] > aabb[a])) return false;
  return true;
}

}  // namespace dfm
}  // namespace ia355
