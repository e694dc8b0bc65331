// The split contractions with the general basis (field basis given as maps;
// the split arithmetic is described in split.hip).  Built, like the
// polynomial adjoint, with the matrix instructions' results in vector
// registers: the phase product's are read by vector instructions at once.
#include "internal.h"
#include "split_dev.h"

namespace expenc {

// One workgroup: 256 rows (64 per wave) x 16 GW columns, over a chunk of the
// other index in tiles of 32.  Forward (ADJ false): rows are samples, own =
// kap, uni = bet; adjoint: rows are pixels, own = bet, uni = kap, the A
// operand exp(+i phi) as well (the conjugation lives in the records).
//
// Phase of tile index k at a row: the FP64 sum of the NT products at the
// centre of the index's 16 (k & ~15) + 8, reduced to [0, 1) turns (the
// anchor), plus the increment sum_j own_j (uni_j(k) - uni_j(centre)) in FP32:
// the differences are taken in FP64 and rounded once, and stay small within
// 16 indexes.  For 32 indexes x 32 rows that is a matrix product of rank NT
// plus one anchor term for each 16 indexes, on v_mfma_f32_32x32x2_f32; the
// differences come as its A operand in lane order (dop[tile][pair of
// terms][lane], zero past NT), the rows' terms as its B operand, once.
// Its output layout (lane: one row, 16 of the tile's indexes) is the
// A-operand layout of the contraction up to a fixed order of the indexes
// inside each 16, in which the records are packed (as for the polynomial
// adjoint).
// Bound: matrix cycles, 1280 of a tile's 2816 for the phase at NT = 17 and
// 32 columns, plus the vector work of sine, cosine and splits.  Before, the
// NT products ran on the vector unit, 16 terms per index by scalar loads:
// their rate bound the kernels (and the adjoint spilled scalar registers).
// Kernel times at 148 x 148, 32 coils, T = 16384, before -> after, measured in turn
// on one card, forward and adjoint: 16 maps fp16 613 -> 405 and 650 -> 428 us, bf16
// 639 -> 407 and 1200 -> 431; 9 maps fp16 437 -> 349 and 617 -> 370, bf16 526 -> 355
// and 586 -> 376.
template <int NT, int GW, bool BF, bool FOLD, bool ADJ>
__global__ __launch_bounds__(256) void k_split_maps(const double *__restrict__ own, const double *__restrict__ uni,
                                                    const float *__restrict__ dop, const u32x4 *__restrict__ rec,
                                                    float *__restrict__ part, const float2 *__restrict__ sq,
                                                    int64_t rows, int64_t K, int NCP, int chunk, int nsplit,
                                                    Bf16Masks mk) {
  constexpr int NJ = (NT + 1) / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int hl = lane >> 5, jl = lane & 31;
  const int nrb = (int)(rows / 256);
  int split, rb;
  if (!(sq ? split_tile_rows(blockIdx.x, nrb, nsplit, &split, &rb) : split_tile(blockIdx.x, nrb, nsplit, &split, &rb)))
    return;
  const int64_t row0 = (int64_t)rb * 256 + wave * 64;
  const int g0 = blockIdx.y * GW;
  const int NGP = NCP / 16;
  const int pz = blockIdx.z;  // problem
  own += pz * rows * NT;
  uni += pz * K * NT;
  dop += pz * K * (2 * NJ);
  rec += pz * K * NGP * 16;
  double pv[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) pv[j] = own[(row0 + lane) * NT + j];
  float bt[2][NJ];
#pragma unroll
  for (int blk = 0; blk < 2; ++blk)
#pragma unroll
    for (int J = 0; J < NJ; ++J) {
      const int j = 2 * J + hl;
      bt[blk][J] = j < NT ? (float)own[(row0 + 32 * blk + jl) * NT + min(j, NT - 1)] : 0.f;
    }
  // A operand of the anchors: term hl belongs to indexes 16 hl .. 16 hl + 15
  const float mine = (jl >> 4) == hl ? 1.f : 0.f;
  f32x16 acc[2][GW];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < GW; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][g][v] = 0.f;
  const int64_t k0 = (int64_t)split * chunk, k1 = min(K, k0 + chunk);
  for (int64_t k = k0; k < k1; k += 32) {
    float a[NJ];
#pragma unroll
    for (int J = NJ - 1; J >= 0; --J) a[J] = dop[((k >> 5) * NJ + J) * 64 + lane];
    const double *u0 = uni + (k + 8) * NT, *u1 = uni + (k + 24) * NT;
    double p0 = 0.0, p1 = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) p0 = fma(pv[j], u0[j], p0);
#pragma unroll
    for (int j = 0; j < NT; ++j) p1 = fma(pv[j], u1[j], p1);
    const auto an = __builtin_amdgcn_permlane32_swap(__float_as_uint((float)__builtin_amdgcn_fract(p0)),
                                                     __float_as_uint((float)__builtin_amdgcn_fract(p1)), false, false);
    f32x16 ph[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int v = 0; v < 16; ++v) ph[blk][v] = 0.f;
    // (last terms first: a basis lists its low orders, the large increments,
    // first, and a sum is rounded at its size with every term that follows)
#pragma unroll
    for (int J = NJ - 1; J >= 0; --J)
#pragma unroll
      for (int blk = 0; blk < 2; ++blk)
        ph[blk] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[J], bt[blk][J], ph[blk], 0, 0, 0);
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
      ph[blk] = __builtin_amdgcn_mfma_f32_32x32x2f32(mine, __uint_as_float(an[blk]), ph[blk], 0, 0, 0);
    // two contraction steps of 16 indexes; ph[blk][8h + i] is index
    // 16h + 8(i/4) + 4hl + i%4 of row jl, K index 8hl + i of step h
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 b[GW][4];
#pragma unroll
      for (int g = 0; g < GW; ++g) {
        const u32x4 *q = rec + (((k >> 4) + h) * NGP + (g0 + g)) * 256 + lane;
        b[g][0] = q[0];
        b[g][1] = q[64];
        b[g][2] = q[128];
        b[g][3] = q[192];
      }
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        u32x4 A[4];  // c hi, c lo, s hi, s lo
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          float c2[2], s2[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float f = __builtin_amdgcn_fractf(ph[blk][8 * h + 2 * m + e]);
            c2[e] = __builtin_amdgcn_cosf(f);
            s2[e] = __builtin_amdgcn_sinf(f);
          }
          uint32_t w[4];
          split_pair<BF>(c2[0], c2[1], w[0], w[1], mk);
          split_pair<BF>(s2[0], s2[1], w[2], w[3], mk);
#pragma unroll
          for (int q = 0; q < 4; ++q) A[q][m] = w[q];
        }
#pragma unroll
        for (int g = 0; g < GW; ++g) acc[blk][g] = step6<BF, FOLD>(A, b[g], acc[blk][g]);
      }
    }
  }
  if constexpr (ADJ)
    adj_epilogue<GW>(part, sq, (int)rows, NCP, nsplit, split, pz, blockIdx.y, gridDim.y, row0, g0, lane, acc);
  else
    store_partials<GW>(part + ((int64_t)pz * nsplit + split) * rows * NCP * 2, row0, NCP, g0, lane, acc, nullptr, 0);
}

template <int NT>
static void launch_maps(const EncPlan &p, const EncBuffers &b, bool adjoint, hipStream_t s) {
  float *part = reinterpret_cast<float *>(b.part);
  const u32x4 *zs = reinterpret_cast<const u32x4 *>(b.zs), *ys = reinterpret_cast<const u32x4 *>(b.ys);
  const Bf16Masks mk = bf16_masks();
  if (adjoint) {
    const dim3 grid(split_grid((int64_t)p.Rp / 256 * p.adj_split), (unsigned)p.NGY, (unsigned)p.P);
    split_variant(p, p.adj_fold, [&](auto gw, auto bf, auto fold) {
      k_split_maps<NT, gw.value, bf.value, fold.value, true><<<grid, 256, 0, s>>>(
          b.bet, b.kap, b.dkap, ys, part, p.comb ? b.sq : nullptr, p.Rp, p.Tp, p.NCP, p.adj_chunk, p.adj_split, mk);
    });
  } else {
    const dim3 grid(split_grid(p.Tp / 256 * p.fwd_split), (unsigned)p.NGY, (unsigned)p.P);
    split_variant(p, [&](auto gw, auto bf) {
      k_split_maps<NT, gw.value, bf.value, false, false><<<grid, 256, 0, s>>>(
          b.kap, b.bet, b.dbet, zs, part, nullptr, p.Tp, p.Rp, p.NCP, p.fwd_chunk, p.fwd_split, mk);
    });
  }
}

void split_maps_launch(const EncPlan &p, const EncBuffers &b, bool adjoint, hipStream_t s) {
  switch (p.NT) {
    case 4: launch_maps<4>(p, b, adjoint, s); break;
    case 10: launch_maps<10>(p, b, adjoint, s); break;
    default: launch_maps<17>(p, b, adjoint, s); break;
  }
}

}  // namespace expenc
