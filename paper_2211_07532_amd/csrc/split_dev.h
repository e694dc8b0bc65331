// Device helpers shared by the split-precision contraction kernels: the
// 16-bit operand types, the hi/lo split of a pair of FP32 values, the 16-bit
// MFMA of either format and the six products of one reduction step.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace expenc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Split two FP32 values into packed (hi, lo) 16-bit pairs.
template <bool BF>
__device__ inline void split_pair(float a, float b, uint32_t &hi, uint32_t &lo) {
  if constexpr (BF) {
    const bf16x2 h = {(__bf16)a, (__bf16)b};
    hi = __builtin_bit_cast(uint32_t, h);
    const float ah = __uint_as_float(hi << 16), bh = __uint_as_float(hi & 0xffff0000u);
    const bf16x2 l = {(__bf16)(a - ah), (__bf16)(b - bh)};
    lo = __builtin_bit_cast(uint32_t, l);
  } else {
    const f16x2 h = {(_Float16)a, (_Float16)b};
    hi = __builtin_bit_cast(uint32_t, h);
    // v - hi in one fused multiply-add that reads the 16-bit half directly
    // (exact: hi is within a factor 2 of v), instead of converting hi back
    // (writing the rounded differences straight into the halves of lo with
    // v_fma_mixlo/mixhi_f16 saves one instruction per pair but measured 1-2 %
    // slower at 1.5 mm)
    float la, lb;
    __asm__("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(la) : "v"(hi), "v"(a));
    __asm__("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(lb) : "v"(hi), "v"(b));
    const f16x2 l = {(_Float16)la, (_Float16)lb};
    lo = __builtin_bit_cast(uint32_t, l);
  }
}

// Masks of the bf16 remainder below, (-1, 0) and (0, -1) as packed bf16
// pairs.  They reach the kernels as arguments (scalar registers): written as
// constants, the compiler encodes (-1, 0) as the inline constant -1.0, which
// the dot-product instruction reads as the FP32 pattern 0xbf800000, (0, -1).
struct Bf16Masks {
  uint32_t lo, hi;
};
inline Bf16Masks bf16_masks() { return Bf16Masks{0x0000bf80u, 0xbf800000u}; }

// split_pair with the bf16 remainders v - hi from a two-term bf16 dot
// product, (hi_a, hi_b) . (-1, 0) + a and (hi_a, hi_b) . (0, -1) + b: one
// instruction per value instead of widening hi and subtracting (exact: the
// product is exact and hi is within a factor 2 of v).  Same bits as
// split_pair<true>; fp16 pairs go to split_pair<false>.
template <bool BF>
__device__ inline void split_pair(float a, float b, uint32_t &hi, uint32_t &lo, Bf16Masks mk) {
  if constexpr (BF) {
    const bf16x2 h = {(__bf16)a, (__bf16)b};
    hi = __builtin_bit_cast(uint32_t, h);
    const float la = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, mk.lo), a, false);
    const float lb = __builtin_amdgcn_fdot2_f32_bf16(h, __builtin_bit_cast(bf16x2, mk.hi), b, false);
    const bf16x2 l = {(__bf16)la, (__bf16)lb};
    lo = __builtin_bit_cast(uint32_t, l);
  } else {
    split_pair<false>(a, b, hi, lo);
  }
}

__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Exact bf16 parts (hi, mid, lo) of two FP32 values of any magnitude.
__device__ inline void split3_any(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  const bf16x2 hv = {(__bf16)a, (__bf16)b};
  h = __builtin_bit_cast(uint32_t, hv);
  const float ra = a - bf16_lo(h), rb = b - bf16_hi(h);
  const bf16x2 mv = {(__bf16)ra, (__bf16)rb};
  m = __builtin_bit_cast(uint32_t, mv);
  const bf16x2 lv = {(__bf16)(ra - bf16_lo(m)), (__bf16)(rb - bf16_hi(m))};
  l = __builtin_bit_cast(uint32_t, lv);
}

template <bool BF>
__device__ inline f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c,
                                                  0, 0, 0);
}

// 6 MFMAs of one step for one 32-row block and one 32-column group:
// cos against b1, sin against b2, each as hi*hi + hi*lo + lo*hi.
template <bool BF>
__device__ inline f32x16 step6(const u32x4 (&A)[4], const u32x4 *b, f32x16 acc) {
  acc = mfma16<BF>(A[0], b[0], acc);
  acc = mfma16<BF>(A[0], b[1], acc);
  acc = mfma16<BF>(A[1], b[0], acc);
  acc = mfma16<BF>(A[2], b[2], acc);
  acc = mfma16<BF>(A[2], b[3], acc);
  acc = mfma16<BF>(A[3], b[2], acc);
  return acc;
}

constexpr int kRec3 = 6 * 64;  // 16-byte words of one FP32-form step and column group

// Operand records of 8 reduction indices (layout: see the packing kernels):
// hi and lo of b1 and b2 (split forms), three exact bf16 parts (FP32 form; o:
// the lane's).
template <bool BF>
__device__ inline void write_record(u32x4 *out, int64_t q, int g, int NGP, int lane, const float (&b1)[8],
                                    const float (&b2)[8]) {
  uint32_t h1[4], l1[4], h2[4], l2[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    split_pair<BF>(b1[2 * m], b1[2 * m + 1], h1[m], l1[m]);
    split_pair<BF>(b2[2 * m], b2[2 * m + 1], h2[m], l2[m]);
  }
  u32x4 *o = out + (q * NGP + g) * 256 + lane;
  o[0] = u32x4{h1[0], h1[1], h1[2], h1[3]};
  o[64] = u32x4{l1[0], l1[1], l1[2], l1[3]};
  o[128] = u32x4{h2[0], h2[1], h2[2], h2[3]};
  o[192] = u32x4{l2[0], l2[1], l2[2], l2[3]};
}

__device__ inline void write_rec3(u32x4 *o, const float (&b1)[8], const float (&b2)[8]) {
  uint32_t w[6][4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    split3_any(b1[2 * m], b1[2 * m + 1], w[0][m], w[1][m], w[2][m]);
    split3_any(b2[2 * m], b2[2 * m + 1], w[3][m], w[4][m], w[5][m]);
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) o[64 * q] = u32x4{w[q][0], w[q][1], w[q][2], w[q][3]};
}

// Writes a wave's forward partial sums; with wmax (scaled form) also the
// wave's max |value| into its slot (a bound for the residual operand), per
// wave and without a workgroup barrier.
template <int GW>
__device__ inline void store_partials(float *dst, int64_t row0, int NCP, int g0, int lane, f32x16 (&acc)[2][GW],
                                      float *wmax, int slot) {
  const int half = lane >> 5, c16 = lane & 15, im = (lane >> 4) & 1;
  float m = 0.f;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int g = 0; g < GW; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t row = row0 + a * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
        const int col = (g0 + g) * 16 + c16;
        dst[(row * NCP + col) * 2 + im] = acc[a][g][v];
        m = fmaxf(m, fabsf(acc[a][g][v]));
      }
  if (wmax) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if (lane == 0) wmax[slot] = m;
  }
}

}  // namespace expenc
