// Device helpers shared by the split-precision contraction kernels: the
// 16-bit operand types, the hi/lo split of a pair of FP32 values, the 16-bit
// MFMA of either format and the six products of one reduction step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

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

// bf16 parts (hi, mid, lo) of two FP32 operand values: exact from 2^-110 (the
// last bit of lo is then at least the smallest bf16, 2^-133) up to the largest
// value, whose hi must not round to infinity.  An infinity or NaN is kept in lo
// alone, which meets no part of the other operand but its hi: one product of
// the right sign, where parts inf, inf - inf give NaN.
__device__ inline void split3_any(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  const bool fa = isfinite(a), fb = isfinite(b);
  constexpr float kMax = 3.38953139e38f;  // the largest bf16
  const bf16x2 hv = {(__bf16)(fa ? fminf(fmaxf(a, -kMax), kMax) : 0.f), (__bf16)(fb ? fminf(fmaxf(b, -kMax), kMax) : 0.f)};
  h = __builtin_bit_cast(uint32_t, hv);
  const float ra = a - bf16_lo(h), rb = b - bf16_hi(h);
  const bf16x2 mv = {(__bf16)(fa ? ra : 0.f), (__bf16)(fb ? rb : 0.f)};
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
// cos against b1, sin against b2, each as hi*hi + hi*lo + lo*hi.  FOLD: the step's
// products start from zero and are added up outside the matrix instruction, which
// rounds a sum that it carries six times a step (EncPlan::fwd_fold).
template <bool BF, bool FOLD>
__device__ inline f32x16 step6(const u32x4 (&A)[4], const u32x4 *b, f32x16 sum) {
  f32x16 acc = FOLD ? f32x16{} : sum;
  acc = mfma16<BF>(A[0], b[0], acc);
  acc = mfma16<BF>(A[0], b[1], acc);
  acc = mfma16<BF>(A[1], b[0], acc);
  acc = mfma16<BF>(A[2], b[2], acc);
  acc = mfma16<BF>(A[2], b[3], acc);
  acc = mfma16<BF>(A[3], b[2], acc);
  return FOLD ? sum + acc : acc;
}

// ---------------------------------------------------------------------------
// Operand scaling of the fp16 and FP32 forms.  An fp16 hi/lo pair represents
// |v| up to 65504 and keeps its ~22-bit precision only while the lo half is
// normal, i.e. for |v| above ~2^-3; three bf16 parts hold all 24 bits from
// 2^-110.  Both forms therefore multiply each packed operand by a power of two
// s = 2^(14 - e), where M < 2^e bounds the operand's magnitudes, so that every
// value lies below 2^14 and values down to 2^-17 (fp16) or 2^-124 (FP32) of the
// largest keep full precision; the reductions that read the contraction's
// output divide s out again (exact for powers of two).
// M comes from a pre-pass over the operand (image operand, or data given at
// the boundary) or from the forward contraction's per-wave output maxima
// (the residual operand, summed over nsplit partial sums).
// ---------------------------------------------------------------------------

__device__ inline float pow2_scale(double m) {
  if (!(m > 0.0) || !isfinite(m)) return 1.f;  // zero, NaN or infinite: unscaled
  int e;
  (void)frexp(m, &e);
  return ldexpf(1.f, min(126, max(-126, 14 - e)));
}

// An element's part in a bound M: |Re| + |Im| (l1) or the larger of the two;
// an element that is not finite has none (its products are not finite at any
// scale, and the other columns keep theirs).
__device__ inline float magnitude(float2 u, bool l1) {
  const float m = l1 ? fabsf(u.x) + fabsf(u.y) : fmaxf(fabsf(u.x), fabsf(u.y));
  return isfinite(u.x) && isfinite(u.y) ? fminf(m, 3.0e38f) : 0.f;
}

// Max of v[0..n) over a 256-thread workgroup; every thread returns it.
__device__ inline float block_max(const float *__restrict__ v, int n) {
  __shared__ float wm[4];
  float m = 0.f;
  int i = threadIdx.x;
  for (; i + 768 < n; i += 1024) {  // four independent loads in flight
    const float a = v[i], b = v[i + 256], c = v[i + 512], d = v[i + 768];
    m = fmaxf(m, fmaxf(fmaxf(a, b), fmaxf(c, d)));
  }
  for (; i < n; i += 256) m = fmaxf(m, v[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  __syncthreads();  // an earlier call's readers are done with wm
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  return fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
}

// Scale of an image operand Z = S u of problem pz from the bounds of u and of
// the coil maps (amax sections 0 and 2 of P problems), both loaded at once.
__device__ inline float image_scale(const float *__restrict__ amax, int pz, int P) {
  __shared__ float wu[4], ws[4];
  const int tid = threadIdx.x;
  static_assert(kAmaxBlocks == 256, "one bound per thread");
  float u = amax[(int64_t)pz * kAmaxBlocks + tid], s = amax[(int64_t)(2 * P + pz) * kAmaxBlocks + tid];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    u = fmaxf(u, __shfl_xor(u, o));
    s = fmaxf(s, __shfl_xor(s, o));
  }
  if ((tid & 63) == 0) {
    wu[tid >> 6] = u;
    ws[tid >> 6] = s;
  }
  __syncthreads();
  return pow2_scale((double)fmaxf(fmaxf(wu[0], wu[1]), fmaxf(wu[2], wu[3])) *
                    fmaxf(fmaxf(ws[0], ws[1]), fmaxf(ws[2], ws[3])));
}

// Scale of a data operand: the bound of the data itself (bnd: its pre-pass)
// or, with nsplit > 0, of the forward's nsplit partial sums (bnd:
// per-wave maxima in units of 1 / inv_z), plus that of the measured data.
__device__ inline float data_scale(const float *__restrict__ bnd, int nbnd, int nsplit, float inv_z,
                                   const float *__restrict__ bnd_meas, int pz) {
  double m = block_max(bnd + (int64_t)pz * nbnd, nbnd);
  if (nsplit > 0) m *= (double)nsplit * inv_z;
  if (bnd_meas) m += block_max(bnd_meas + (int64_t)pz * kAmaxBlocks, kAmaxBlocks);
  return pow2_scale(m);
}

// go(GW, BF) for a split plan, and go(GW, BF, FOLD)
template <class Go>
inline void split_variant(const EncPlan &p, Go go) {
  auto width = [&](auto bf) {
    if (p.GW == 2) go(std::integral_constant<int, 2>{}, bf);
    else go(std::integral_constant<int, 1>{}, bf);
  };
  if (p.prec == EXPENC_BF16_SPLIT) width(std::true_type{});
  else width(std::false_type{});
}
template <class Go>
inline void split_variant(const EncPlan &p, bool fold, Go go) {
  if (fold) split_variant(p, [&](auto gw, auto bf) { go(gw, bf, std::true_type{}); });
  else split_variant(p, [&](auto gw, auto bf) { go(gw, bf, std::false_type{}); });
}

constexpr int kRec3 = 6 * 64;  // 16-byte words of one FP32-form step and column group

// Operand records of 8 reduction indices (layout: see the packing kernels):
// hi and lo of b1 and b2 (split forms), three bf16 parts (FP32 form; o: the
// lane's).
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
