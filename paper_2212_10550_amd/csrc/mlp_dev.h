// The decoder MLP of Sec. 3.1, Eq. 1-2 (32 -> 64 -> 64 -> 4) in its BF16
// MFMA form (internal).  Layouts: see mlp.hip.  The decoder forward and the
// persistent batch renderer share everything here but the chain of layers
// (several tiles against one): the same operations in the same order, which
// the batch tests hold to the same bits.
#pragma once
#include <hip/hip_bf16.h>

#include "common.h"

namespace ia355 {
namespace mlpd {

constexpr int NIN = 32, NH = 64, NOUT = 4;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NIN, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NOUT * NH, NPARAM = OFF_B3 + NOUT;
static_assert(NPARAM == 6532, "parameter count");

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// max(z, 0) as a signed-integer max of the bits: one v_max_i32 (fmaxf
// first quiets its MFMA-produced input, a second instruction).  Every
// non-negative float keeps its bits, every negative one (and -0) gives +0;
// a NaN with the sign bit clear propagates.
__device__ __forceinline__ float relu(float z) {
  const int b = __builtin_bit_cast(int, z);
  return __builtin_bit_cast(float, b > 0 ? b : 0);
}

// Density exp(o0) (clamped at exp(80)) and colour sigmoid(o1..3); the
// sigmoid's reciprocal is the hardware one (1 ulp), not a division.
__device__ __forceinline__ void head(const float o[4], float *sig, float c[3]) {
  *sig = expf(fminf(o[0], 80.0f));
#pragma unroll
  for (int k = 0; k < 3; ++k) c[k] = __builtin_amdgcn_rcpf(1.0f + expf(-o[1 + k]));
}

// --------------------------------------------------------------- BF16 fwd
// Parameter index of element j of lane (r, g)'s fragments (-1: zero).
__host__ __device__ inline int w1_at(int mt, int r, int g, int j) { return OFF_W1 + (16 * mt + r) * NIN + 8 * g + j; }
__host__ __device__ inline int w2_at(int mt, int c, int r, int g, int j) {
  return OFF_W2 + (16 * mt + r) * NH + 16 * (2 * c + j / 4) + 4 * g + (j % 4);
}
__host__ __device__ inline int w3_at(int c, int r, int g, int j) {
  return r < NOUT ? OFF_W3 + r * NH + 16 * (2 * c + j / 4) + 4 * g + (j % 4) : -1;
}
__device__ __forceinline__ __bf16 frag_value(const float *P, int i) { return (__bf16)(i >= 0 ? P[i] : 0.0f); }

// Fragment q (0-3: w1[q], 4-11: w2[(q-4)/2][(q-4)%2], 12-13: w3[q-12]) of
// lane (r, g).
__device__ __forceinline__ bf16x8 frag_bf(const float *P, int q, int r, int g) {
  bf16x8 v;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int i = q < 4 ? w1_at(q, r, g, j) : (q < 12 ? w2_at((q - 4) / 2, (q - 4) % 2, r, g, j) : w3_at(q - 12, r, g, j));
    v[j] = frag_value(P, i);
  }
  return v;
}

// First parameter of half h (elements 4h .. 4h + 3, consecutive parameters)
// of fragment q of lane (r, g); -1: a zero half.
__host__ __device__ inline int frag_half_at(int q, int r, int g, int h) {
  return q < 4 ? w1_at(q, r, g, 4 * h) : (q < 12 ? w2_at((q - 4) / 2, (q - 4) % 2, r, g, 4 * h) : w3_at(q - 12, r, g, 4 * h));
}

// The BF16 decoder's fragments in LDS, one 16-byte slot per lane so that a
// wave reads a fragment with one conflict-free load: mw[q][lane] holds
// fragment q (0-3 layer 1, 4 + 2 mt + c layer 2, 12 + c layer 3) of lane
// (lane % 16, lane / 16); b1, b2, b3 the biases.
struct FragLds {
  bf16x8 mw[14][64];
  float b1[NH], b2[NH], b3[NOUT];
};
static_assert(offsetof(FragLds, b1) % 16 == 0 && offsetof(FragLds, b2) % 16 == 0 && offsetof(FragLds, b3) % 16 == 0,
              "16-byte bias vectors");

// Weights fetched from a FragLds as each MFMA needs them.
struct LdsW {
  const FragLds &s;
  int lane, g;
  __device__ __forceinline__ bf16x8 w1(int mt) const { return s.mw[mt][lane]; }
  __device__ __forceinline__ bf16x8 w2(int mt, int c) const { return s.mw[4 + 2 * mt + c][lane]; }
  __device__ __forceinline__ bf16x8 w3(int c) const { return s.mw[12 + c][lane]; }
  __device__ __forceinline__ f32x4 b1(int mt) const { return *reinterpret_cast<const f32x4 *>(s.b1 + 16 * mt + 4 * g); }
  __device__ __forceinline__ f32x4 b2(int mt) const { return *reinterpret_cast<const f32x4 *>(s.b2 + 16 * mt + 4 * g); }
};

// A compiler-only barrier inside a loop: the LDS fragment reads after it
// cannot be hoisted out of the loop (which would hold every fragment in
// registers again).
__device__ __forceinline__ void pin_in_loop() { asm volatile("" ::: "memory"); }

// Pack the relu'd accumulators of tiles t = 2c, 2c+1 into one B operand.
__device__ __forceinline__ bf16x8 pack_act(const f32x4 z[4], int c) {
  bf16x8 b;
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = (__bf16)relu(z[2 * c + j / 4][j % 4]);
  return b;
}

// The BF16 forward of one 16-sample tile with the weights from a source:
// w.w1(mt), w.w2(mt, c), w.w3(c) give the A-operand fragments and w.b1(mt),
// w.b2(mt), w.b3() the accumulator initialisers (biases).
template <class WSrc>
__device__ __forceinline__ void fwd_bf_src(const WSrc &w, const bf16x8 &X, f32x4 z1[4], f32x4 z2[4], f32x4 &o) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) z1[mt] = mfma32(w.w1(mt), X, w.b1(mt));
  const bf16x8 h1a = pack_act(z1, 0), h1b = pack_act(z1, 1);
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    f32x4 acc = w.b2(mt);
    acc = mfma32(w.w2(mt, 0), h1a, acc);
    z2[mt] = mfma32(w.w2(mt, 1), h1b, acc);
  }
  const bf16x8 h2a = pack_act(z2, 0), h2b = pack_act(z2, 1);
  f32x4 acc = w.b3();
  acc = mfma32(w.w3(0), h2a, acc);
  o = mfma32(w.w3(1), h2b, acc);
}

}  // namespace mlpd
}  // namespace ia355
