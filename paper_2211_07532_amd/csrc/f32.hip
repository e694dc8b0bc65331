// FP32 form of the encoding contractions, on the bf16 matrix cores.
//
// Every FP32 operand value is written as hi + mid + lo with hi = rnd(v),
// mid = rnd(v - hi) and lo = v - hi - mid in bf16: three 8-bit significands
// hold the 24 bits of v exactly, where lo's last bit is a bf16 value (from
// 2^-110; operands are packed times a power of two, split_dev.h).  A product a*b is taken as
//   a_hi b_hi + a_hi b_mid + a_mid b_hi + a_hi b_lo + a_lo b_hi + a_mid b_mid
// on v_mfma_f32_32x32x16_bf16 with FP32 accumulation; the three products left
// out are below 2^-25 of it, under the rounding of one FP32 addition.  Phases
// are FP64 throughout, as the field may be of any strength.
//
// Why: v_mfma_f32_32x32x2_f32 takes 4096 matrix cycles per 16 reduction
// indices, 64 rows and 32 columns, the six bf16 products 1536, for a few
// hundred cycles more of vector work (three splits, the exchanges); neither
// overlaps much with the FP64 phase.  Kernel times at 148 x 148, 32 coils, T =
// 16384, on the FP32 instruction and now, measured in turn on one card, forward /
// adjoint: solid harmonics 960 / 1107 -> 612 / 650 us, 16 maps 1031 / 1165 -> 793 /
// 783 us, 9 maps 903 / 1019 -> 659 / 689 us.  Bound: matrix cycles plus the
// vector work of the phase, sine, cosine and splits.  The error against FP64
// does not grow (adjoint 200 x 200, 32 coils, T = 40000: 4.8e-7 -> 3.0e-7).
//
// A sum carried through the matrix instruction loses the more the larger it has
// grown, always to the same side (split_sign), and is rounded twelve times a
// step.  With FOLD every step's products start from zero and the result is added
// to the accumulators outside.  These sums are the more precise ones, which lets
// small problems have chunks of 64 where they had 16 (make_plan); on long chunks
// it costs 6 to 45 % (16 to 64 more registers, no overlap of a step's last
// products with the next phases).
// Error of the adjoint of random data relative to the FP32 instruction's, without
// signs and folds and now: 148 x 148, 32 coils, T = 16384 1.53 -> 0.83, 128 x 128,
// 16 coils, T = 12000 1.14 -> 0.84, 40 x 33, 8 coils, T = 3000 (64 samples against
// 16) 1.36 -> 0.82.
//
// Layout of one step (K = 16 reduction indices) as in the split forms: lane l
// holds indices 8*(l/32) .. +7 of row l%32 (A) or column l%32 (B).  Each lane
// evaluates its OWN row against 16 wave-uniform indices, splits and packs
// pairs, and v_permlane32_swap exchanges the half-waves, so that the two
// 32-row blocks of the wave get their operands.  The B operand is packed in
// lane order: six 16-byte records per lane and step (b1 hi, mid, lo, b2 hi,
// mid, lo; b1 against cos, b2 against sin).
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "internal.h"
#include "split_dev.h"

namespace expenc {

// (hi, mid, lo) pairs of two FP32 values (exact remainders: the bf16 dot
// product v + (hi_a, hi_b) . (-1, 0), see split_pair).
__device__ inline void split3(float a, float b, Bf16Masks mk, uint32_t &h, uint32_t &m, uint32_t &l) {
  const bf16x2 ma = __builtin_bit_cast(bf16x2, mk.lo), mb = __builtin_bit_cast(bf16x2, mk.hi);
  const bf16x2 hv = {(__bf16)a, (__bf16)b};
  const float ra = __builtin_amdgcn_fdot2_f32_bf16(hv, ma, a, false);
  const float rb = __builtin_amdgcn_fdot2_f32_bf16(hv, mb, b, false);
  const bf16x2 mv = {(__bf16)ra, (__bf16)rb};
  const float la = __builtin_amdgcn_fdot2_f32_bf16(mv, ma, ra, false);
  const float lb = __builtin_amdgcn_fdot2_f32_bf16(mv, mb, rb, false);
  const bf16x2 lv = {(__bf16)la, (__bf16)lb};
  h = __builtin_bit_cast(uint32_t, hv);
  m = __builtin_bit_cast(uint32_t, mv);
  l = __builtin_bit_cast(uint32_t, lv);
}

// A phase in turns (FP64), reduced to [-1/2, 1/2] before it is rounded to FP32
__device__ inline float reduce_turns(double p) { return (float)(p - __builtin_rint(p)); }

__device__ inline void sincos_turns(double p, float &c, float &s) {
  const float f = reduce_turns(p);
  c = __builtin_amdgcn_cosf(f);
  s = __builtin_amdgcn_sinf(f);
}

// The six products of cos against b1 and of sin against b2, smallest first.
// A: [c hi, c mid, c lo, s hi, s mid, s lo].
template <bool FOLD>
__device__ inline f32x16 step12(const u32x4 (&A)[6], const u32x4 (&b)[6], f32x16 sum) {
  f32x16 acc = FOLD ? f32x16{} : sum;
#pragma unroll
  for (int o = 0; o < 6; o += 3) {
    acc = mfma16<true>(A[o + 1], b[o + 1], acc);
    acc = mfma16<true>(A[o + 2], b[o], acc);
    acc = mfma16<true>(A[o], b[o + 2], acc);
    acc = mfma16<true>(A[o + 1], b[o], acc);
    acc = mfma16<true>(A[o], b[o + 1], acc);
    acc = mfma16<true>(A[o], b[o], acc);
  }
  return FOLD ? sum + acc : acc;
}

// Wave-uniform terms of one reduction index (scalar loads).  The opaque
// offset keeps the loads of one index from being merged with or hoisted above
// those of an earlier one: two indices' terms are live at a time.
template <int NU>
__device__ inline void load_uniform(const double *__restrict__ u, int off, double (&q)[NU]) {
  __asm__ volatile("" : "+s"(off));
#pragma unroll
  for (int j = 0; j < NU; ++j) q[j] = u[off + j];
}

struct F32Args {
  int64_t Tp;
  int Rp, NCP, NGP, chunk, nsplit, nxq, nx, ny, pix0;  // NGP, Rp, pix0: groups, pixels and first pixel of a pass
  double dx, dy;
  Bf16Masks mk;
  float *wmax;  // forward: per-wave maxima of the partial sums
};

// Exchanges the packed words of the lane's own row (w[kind][pair], pairs of
// reduction indices) into the two blocks' operands and adds the step's
// products; o: the step's records of the first column group, this lane's.
template <int GW, bool FOLD>
__device__ inline void contract16(const uint32_t (&w)[6][8], const u32x4 *__restrict__ o, f32x16 (&acc)[2][GW]) {
  u32x4 A[2][6];
#pragma unroll
  for (int q = 0; q < 6; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const auto r = __builtin_amdgcn_permlane32_swap(w[q][i], w[q][4 + i], false, false);
      A[0][q][i] = r[0];
      A[1][q][i] = r[1];
    }
#pragma unroll
  for (int g = 0; g < GW; ++g) {
    const u32x4 *og = o + g * kRec3;
    const u32x4 b[6] = {og[0], og[64], og[128], og[192], og[256], og[320]};
    acc[0][g] = step12<FOLD>(A[0], b, acc[0][g]);
    acc[1][g] = step12<FOLD>(A[1], b, acc[1][g]);
  }
}

template <int GW>
__device__ inline void zero_acc(f32x16 (&acc)[2][GW]) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int g = 0; g < GW; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[b][g][v] = 0.f;
}

// Software pipeline of the solid-harmonic forward: the products of one step
// are issued between the vector work of the next step's phases.  A group's
// records follow in halves (cos, sin) as soon as the half before is used up.
// 32 coils: 5.5 % less time at 148 x 148, T = 16384, 6.3 % at 200 x 200, T = 20000
// (one column group: equal).  The adjoint, which waits for its LDS reads as well,
// took 3 % more with the same pipeline.
template <int GW, bool FOLD>
struct Pipe {
  static constexpr int N = 24 * GW;  // MFMAs of a step
  u32x4 A[2][6], b[6];
  f32x16 t[2];       // FOLD: a column group's sums over the step
  uint32_t w[6][8];  // the next step's words, as for contract16

  __device__ inline void load(int h, const u32x4 *__restrict__ rec) {
#pragma unroll
    for (int q = 0; q < 3; ++q) b[3 * h + q] = rec[64 * (3 * h + q)];
  }
  // the words of a pair of indices (phases in turns, reduced)
  __device__ inline void pair(int m, float f0, float f1, Bf16Masks mk) {
    split3(__builtin_amdgcn_cosf(f0), __builtin_amdgcn_cosf(f1), mk, w[0][m], w[1][m], w[2][m]);
    split3(__builtin_amdgcn_sinf(f0), __builtin_amdgcn_sinf(f1), mk, w[3][m], w[4][m], w[5][m]);
  }
  __device__ inline void exchange() {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(w[q][i], w[q][4 + i], false, false);
        A[0][q][i] = r[0];
        A[1][q][i] = r[1];
      }
  }
  // MFMAs [lo, hi) of the step: groups in turn, cos then sin, step12's order
  // for each row block, the blocks alternating; cur, next: this lane's records
  // of the step and of the one after
  __device__ inline void products(int lo, int hi, const u32x4 *__restrict__ cur, const u32x4 *__restrict__ next,
                                  f32x16 (&acc)[2][GW]) {
    constexpr int pa[6] = {1, 2, 0, 1, 0, 0}, pb[6] = {1, 0, 2, 0, 1, 0};
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (k >= lo && k < hi) {
        const int g = k / 24, h = k % 24 / 12, q = k % 12 >> 1, blk = k & 1;
        f32x16 &c = FOLD ? t[blk] : acc[blk][g];
        if (FOLD && k % 24 < 2) c = f32x16{};
        c = mfma16<true>(A[blk][3 * h + pa[q]], b[3 * h + pb[q]], c);
        if (FOLD && k % 24 >= 22) acc[blk][g] += c;
        if (k % 12 == 11) load(h, g + 1 < GW ? cur + (g + 1) * kRec3 : next);
      }
  }
};

// One workgroup: 256 rows (64 per wave) x 16 GW columns x a chunk of the
// reduction.  FWD: rows are samples, the reduction runs over pixels; else
// rows are pixels and it runs over samples.  NT: terms of the general basis
// (17 FP64 products an entry at L = 16), or 0 (forward) for the solid
// harmonics: along a 16-pixel tile of an image row a sample's phase is a
// cubic (coefficients from the row polynomial at the tile's centre; pixels at
// equal distances from it share their even and odd parts, so 2 FP64 products an
// entry and one for the off-resonance).
// own, uni: the rows' terms [rows][NT] and the reduction indices' terms
// [n][NT] of the general basis, or pmono and dwq; opr: operand records.
// (restrict kernel arguments: uniform terms become scalar loads)
// The reduction indices' first lds_terms(NT) terms go through LDS (blocks of
// kIndices, double-buffered, one barrier per block) and the rest through the
// scalar cache: with 17 FP64 terms an index the scalar cache's fills bound the
// kernel, and a broadcast read costs the LDS a full one.  Time at 148 x 148, 32
// coils, T = 16384 relative to that with 6 terms in LDS, forward / adjoint: none
// 1.38 / 1.43, 4 1.02 / 1.03, 8 1.13 / 1.16; 10 terms an index fit the scalar path
// alone (with 4 to 6 in LDS 1.04 / 1.03 of the time).
constexpr int kIndices = 64;
constexpr int lds_terms(int nt) { return nt == 17 ? 6 : 0; }

template <int NT, int GW, bool FWD, bool FOLD>
__device__ inline void f32_body(const double *__restrict__ own, const double *__restrict__ uni,
                                const u32x4 *__restrict__ opr, float *__restrict__ part, const F32Args &a) {
  static_assert(NT || FWD, "the solid-harmonic adjoint is k_adj_f32_sh");
  constexpr int NL = lds_terms(NT), NS = NT - NL;
  __shared__ double sh[2][NL ? kIndices : 1][NL ? NL : 2];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t rows = FWD ? a.Tp : a.Rp, len = FWD ? a.Rp : a.Tp;
  int split, rb;
  const int pz = blockIdx.z;  // problem
  auto wmax = [&] {  // this wave's slot
    return FWD ? a.wmax + ((int64_t)(pz * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * 4 + wave : nullptr;
  };
  if (!split_tile(blockIdx.x, (int)(rows / 256), a.nsplit, &split, &rb)) {
    if (FWD && lane == 0) *wmax() = 0.f;
    return;
  }
  const int64_t row0 = (int64_t)rb * 256 + wave * 64;
  const int g0 = blockIdx.y * GW;
  const int NGP = a.NGP;
  constexpr int NP = NT ? NT : 11;
  constexpr int S = NT ? NT : kPolyStride;  // row strides of the tables
  own += pz * (NT ? rows : a.Tp) * S;
  uni += NT ? pz * len * S : (int64_t)pz * a.Rp;
  const u32x4 *__restrict__ op = opr + ((int64_t)pz * (len / 16) * NGP + g0) * kRec3 + lane;
  double P[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) P[j] = own[(row0 + lane) * S + j];
  f32x16 acc[2][GW];
  zero_acc<GW>(acc);
  const int64_t k0 = (int64_t)split * a.chunk;
  const int64_t k1 = min(len, k0 + a.chunk);
  const double dx2 = a.dx * a.dx, dx3 = dx2 * a.dx;
  auto fill = [&](int64_t kb, int buf) {
    const int n = (int)min<int64_t>(kIndices, k1 - kb) * NL;
    for (int i = threadIdx.x; i < n; i += 256) (&sh[buf][0][0])[i] = uni[(kb + i / NL) * S + i % NL];
  };
  if constexpr (NL > 0) {
    fill(k0, 0);
    __syncthreads();
  }
  if constexpr (NT == 0) {
    Pipe<GW, FOLD> pp;
    RowCubic rc;
    rc.start(a.pix0 + (int)k0, a.nxq);
    float f[16];
    const int64_t step = (int64_t)NGP * kRec3;
    const u32x4 *__restrict__ cur = op + (k0 >> 4) * step;
    auto phase = [&](int r, int m) {  // pixels 8 + m and 8 - m (m = 0: 8 and 0)
      double lo, hi;
      rc.two(m, lo, hi);
      f[(8 - m) & 7] = reduce_turns(fma(P[10], uni[r + ((8 - m) & 7)], lo));
      f[8 + m] = reduce_turns(fma(P[10], uni[r + 8 + m], hi));
    };
    pp.load(0, cur);
    pp.load(1, cur);
    rc.expand(P, a.nx, a.ny, a.dx, a.dy, dx2, dx3);
    rc.next(a.nxq);
#pragma unroll
    for (int m = 0; m < 8; ++m) phase((int)k0, m);
#pragma unroll
    for (int m = 0; m < 8; ++m) pp.pair(m, f[2 * m], f[2 * m + 1], a.mk);
    pp.exchange();
    for (int64_t k = k0; k + 16 < k1; k += 16, cur += step) {
      constexpr int N = Pipe<GW, FOLD>::N;
      rc.expand(P, a.nx, a.ny, a.dx, a.dy, dx2, dx3);
      rc.next(a.nxq);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        pp.products(N * m / 16, N * (m + 1) / 16, cur, cur + step, acc);
        phase((int)k + 16, m);
      }
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        pp.products(N * (m + 8) / 16, N * (m + 9) / 16, cur, cur + step, acc);
        pp.pair(m, f[2 * m], f[2 * m + 1], a.mk);
      }
      pp.exchange();
    }
    pp.products(0, Pipe<GW, FOLD>::N, cur, cur, acc);
  } else {
    for (int64_t k = k0; k < k1; k += 16) {
      uint32_t w[6][8];  // [c hi, mid, lo, s hi, mid, lo][pair of the 16 indices]
      const int in = (int)(k - k0) & (kIndices - 1), buf = (int)((k - k0) / kIndices) & 1;
      if constexpr (NL > 0) {
        if (in == 0 && k + kIndices < k1) fill(k + kIndices, buf ^ 1);
      }
      // the 16 indices' scalar terms, loaded one index ahead of their use
      const double *u0 = uni + k * S + NL;
      double q[2][NS];
      load_uniform<NS>(u0, 0, q[0]);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        float c[2], s[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int i = 2 * m + e;
          if (i < 15) load_uniform<NS>(u0, (i + 1) * S, q[(i + 1) & 1]);
          double p = 0.0;
#pragma unroll
          for (int j = 0; j < NL; ++j) p = fma(sh[buf][NL ? in + i : 0][j], P[j], p);
#pragma unroll
          for (int j = 0; j < NS; ++j) p = fma(q[e][j], P[NL + j], p);
          sincos_turns(p, c[e], s[e]);
        }
        split3(c[0], c[1], a.mk, w[0][m], w[1][m], w[2][m]);
        split3(s[0], s[1], a.mk, w[3][m], w[4][m], w[5][m]);
      }
      contract16<GW, FOLD>(w, op + (k >> 4) * NGP * kRec3, acc);
      if constexpr (NL > 0) {
        if (((k - k0) & (kIndices - 1)) == kIndices - 16) __syncthreads();
      }
    }
  }
  // [problem][split][row][column] complex
  store_partials<GW>(part + ((int64_t)pz * a.nsplit + split) * rows * a.NCP * 2, row0, a.NCP, g0, lane, acc, wmax(),
                     0);
}

// Waves per SIMD asked for: 17 terms and 32 columns need 169 registers left to
// the compiler, one more than three waves have (148 x 148, 32 coils, T = 16384
// forward: two waves take 1.14 times as long).
constexpr int min_waves(int nt, int gw, bool fold) { return nt == 17 && gw == 2 && !fold ? 3 : 2; }

template <int NT, int GW, bool FOLD>
__global__ __launch_bounds__(256, min_waves(NT, GW, FOLD)) void k_fwd_f32(const double *__restrict__ own, const double *__restrict__ uni,
                                                     const u32x4 *__restrict__ op, float *__restrict__ part,
                                                     F32Args a) {
  f32_body<NT, GW, true, FOLD>(own, uni, op, part, a);
}

template <int NT, int GW, bool FOLD>
__global__ __launch_bounds__(256, min_waves(NT, GW, FOLD)) void k_adj_f32(const double *__restrict__ own, const double *__restrict__ uni,
                                                     const u32x4 *__restrict__ op, float *__restrict__ part,
                                                     F32Args a) {
  f32_body<NT, GW, false, FOLD>(own, uni, op, part, a);
}

// The solid-harmonic adjoint (rows: pixels, reduction over samples).  At a
// pixel (x, y) sample t has the phase
//   a_0 + x (a_1 + x (a_2 + x a_3)) + t dw0,
// a_j polynomials in y with the sample's coefficients.  A workgroup's 256
// pixels lie in a few image rows, so it evaluates the a_j of kSamples samples
// at those rows into LDS (double-buffered, one barrier per block of samples)
// and a lane reads its row's four and t: 4 FP64 products an entry and 40
// bytes from LDS (broadcast within a row).  With the sample's ten
// coefficients as scalar operands it took 10 products, and the scalar cache's
// fills bound it: 1.18 times the time at 148 x 148, 32 coils, T = 16384.
constexpr int kSamples = 64;

template <int GW, bool FOLD>
__global__ __launch_bounds__(256, 2) void k_adj_f32_sh(const double *__restrict__ pmono,
                                                       const double *__restrict__ dwq,
                                                       const u32x4 *__restrict__ opr, float *__restrict__ part,
                                                       F32Args a, int nrow) {
  extern __shared__ double sh[];  // [2][kSamples][nrow][4], then t [2][kSamples]
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int split, rb;
  if (!split_tile(blockIdx.x, a.Rp / 256, a.nsplit, &split, &rb)) return;
  const int64_t row0 = (int64_t)rb * 256 + wave * 64;
  const int g0 = blockIdx.y * GW;
  const int NGP = a.NCP / 16;
  const int pz = blockIdx.z;  // problem
  pmono += pz * a.Tp * kPolyStride;
  dwq += (int64_t)pz * a.Rp;
  const u32x4 *__restrict__ op = opr + ((int64_t)pz * (a.Tp / 16) * NGP + g0) * kRec3 + lane;
  const int rq = (int)row0 + lane, yfirst = rb * 256 / a.nxq;
  const double x = (rq % a.nxq - 0.5 * a.nx) * a.dx, w0 = dwq[rq];
  double *const tt = sh + 2 * kSamples * nrow * 4;
  const int64_t k0 = (int64_t)split * a.chunk, k1 = min(a.Tp, k0 + a.chunk);
  auto fill = [&](int64_t kb, int buf) {
    const int ns = (int)min<int64_t>(kSamples, k1 - kb);
    for (int i = threadIdx.x; i < ns * nrow; i += 256) {
      const int j = i / nrow, r = i - j * nrow;
      const double *P = pmono + (kb + j) * kPolyStride;
      const double y = (yfirst + r - 0.5 * a.ny) * a.dy;
      double *o = sh + ((buf * kSamples + j) * nrow + r) * 4;
      o[0] = fma(y, fma(y, fma(y, P[9], P[5]), P[2]), P[0]);
      o[1] = fma(y, fma(y, P[8], P[4]), P[1]);
      o[2] = fma(y, P[7], P[3]);
      o[3] = P[6];
      if (r == 0) tt[buf * kSamples + j] = P[10];
    }
  };
  f32x16 acc[2][GW];
  zero_acc<GW>(acc);
  fill(k0, 0);
  __syncthreads();
  int buf = 0;
  for (int64_t kb = k0; kb < k1; kb += kSamples, buf ^= 1) {
    if (kb + kSamples < k1) fill(kb + kSamples, buf ^ 1);
    const int ns = (int)min<int64_t>(kSamples, k1 - kb);
    const double2 *cf = reinterpret_cast<const double2 *>(sh) + (buf * kSamples * nrow + rq / a.nxq - yfirst) * 2;
    const double *ct = tt + buf * kSamples;
    for (int j0 = 0; j0 < ns; j0 += 16) {
      uint32_t w[6][8];  // [c hi, mid, lo, s hi, mid, lo][pair of the 16 indices]
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        float c[2], s[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int j = j0 + 2 * m + e;
          const double2 a01 = cf[j * nrow * 2], a23 = cf[j * nrow * 2 + 1];
          sincos_turns(fma(ct[j], w0, fma(x, fma(x, fma(x, a23.y, a23.x), a01.y), a01.x)), c[e], s[e]);
        }
        split3(c[0], c[1], a.mk, w[0][m], w[1][m], w[2][m]);
        split3(s[0], s[1], a.mk, w[3][m], w[4][m], w[5][m]);
      }
      contract16<GW, FOLD>(w, op + ((kb + j0) >> 4) * NGP * kRec3, acc);
    }
    __syncthreads();
  }
  adj_epilogue<GW>(part, nullptr, a.Rp, a.NCP, a.nsplit, split, pz, blockIdx.y, gridDim.y, row0, g0, lane, acc);
}

// ---------------------------------------------------------------------------
// Operand packing.  Record (step q, group g, lane l): 8 reduction indices
// 16q + 8*(l/32) + i, column col = 16g + l%16, part = (l/16)&1.
//   forward:  b1 = part ? Zi : Zr,   b2 = part ? Zr : -Zi
//   adjoint:  b1 = part ? Yi : Yr,   b2 = part ? -Yr : Yi
// times the operand's scale and the sign of the index's split.
// ---------------------------------------------------------------------------

// Z[r'][col] = S_c(r) x_b(r), col = b*C + c, row r' = y*nxq + x of pixel
// r = y*nx + x; zero for padded pixels and columns.  npix pixels from pix0 on and
// NGP column groups from gf on (a pass, or all).
__global__ __launch_bounds__(256) void k_build_z_f32(const float2 *__restrict__ smaps, const float2 *__restrict__ x,
                                                     int64_t x_stride, int x_row_stride, int nx, int ny, int nxq,
                                                     int npix, int pix0, int C, int NC, int gf, int NGP,
                                                     u32x4 *__restrict__ zs, int64_t x_pstride, int chunk,
                                                     const float *__restrict__ amax,
                                                     float *__restrict__ scl) {
  const int R = nx * ny;
  const int64_t pz = blockIdx.y;
  int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = id < (int64_t)(npix / 16) * NGP * 64;
  if (!live) id = 0;
  const int lane = (int)(id & 63);
  const int64_t qg = id >> 6;
  const int g = gf + (int)(qg % NGP);
  const int col = 16 * g + (lane & 15), im = (lane >> 4) & 1;
  const int rq0 = pix0 + (int)(16 * (qg / NGP) + 8 * (lane >> 5));
  int yy = rq0 / nxq, xx = rq0 - yy * nxq;
  const bool colok = col < NC;
  const int b = colok ? col / C : 0, c = colok ? col % C : 0;
  smaps += (pz * C + c) * R;
  x += pz * x_pstride + b * x_stride;
  float2 u[8], s[8];
  bool ok[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    ok[i] = yy < ny && xx < nx && colok;
    const int yc = ok[i] ? yy : 0, xc = ok[i] ? xx : 0;
    u[i] = x[(int64_t)yc * x_row_stride + xc];
    s[i] = smaps[yc * nx + xc];
    if (++xx == nxq) {
      xx = 0;
      ++yy;
    }
  }
  // (every workgroup derives the same power of two, behind its loads)
  const float sc = image_scale(amax, (int)pz, gridDim.y);
  if (blockIdx.x == 0 && threadIdx.x == 0) scl[2 * pz] = sc;
  if (!live) return;
  const float f = sc * split_sign((pix0 + 16 * (qg / NGP)) / chunk);
  float b1[8], b2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float2 z = ok[i] ? make_float2((s[i].x * u[i].x - s[i].y * u[i].y) * f,
                                         (s[i].x * u[i].y + s[i].y * u[i].x) * f)
                           : make_float2(0.f, 0.f);
    b1[i] = im ? z.y : z.x;
    b2[i] = im ? z.x : -z.y;
  }
  write_rec3(zs + (pz * (npix / 16) * NGP + qg) * kRec3 + lane, b1, b2);
}

// Adjoint operand: sign * y, y [B][T][C] (src), or the forward's partial sums
// (part, added in FP64 in the order of the splits, their signs undone) minus y_meas (may be
// NULL).  Padded rows and columns are zero.  The residual is also kept as
// yop [Tp][NCP] (its norm is the Rayleigh quotient and the data term).
__global__ __launch_bounds__(256) void k_pack_y_f32(const float2 *__restrict__ src, float sign, int chunk,
                                                    const float2 *__restrict__ part, int nsplit,
                                                    const float2 *__restrict__ y_meas, int64_t T, int64_t Tp, int C,
                                                    int NC, int NCP, u32x4 *__restrict__ ys,
                                                    float2 *__restrict__ yop, const float *__restrict__ bnd, int nbnd,
                                                    const float *__restrict__ bnd_meas, float *__restrict__ scl) {
  const int NGP = NCP / 16;
  const int64_t pz = blockIdx.y;
  const float inv_z = src ? 1.f : 1.f / scl[2 * pz];
  int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = id < (Tp / 16) * NGP * 64;
  if (!live) id = 0;
  const int lane = (int)(id & 63);
  const int64_t qg = id >> 6;
  const int col = 16 * (int)(qg % NGP) + (lane & 15), im = (lane >> 4) & 1;
  const int64_t t0 = 16 * (qg / NGP) + 8 * (lane >> 5);
  const int b = col / C, c = col % C;
  float2 y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) y[i] = make_float2(0.f, 0.f);
  // (loads of padded samples repeat the last: under a branch each waits alone)
  const float2 *data = src ? src : y_meas;
  float2 m[8];
  if (data && col < NC) {
#pragma unroll
    for (int i = 0; i < 8; ++i) m[i] = data[((pz * NC / C + b) * T + min(t0 + i, T - 1)) * C + c];
  }
  if (src) {
    if (col < NC) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (t0 + i < T) y[i] = make_float2(sign * m[i].x, sign * m[i].y);
    }
  } else if (col < NC) {
    double sx[8], sy[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sx[i] = sy[i] = 0.0;
    const float2 *p = part + (pz * nsplit * Tp + t0) * NCP + col;
    // four splits' loads together, the last split repeated at the end: with one
    // split at a time and y_meas under branches 20 us, so 18 (55 x 27, 10 coils,
    // T 2875, 48 splits, 48 workgroups)
    for (int k = 0; k < nsplit; k += 4) {
      float2 v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) v[u][i] = p[(min(k + u, nsplit - 1) * Tp + i) * NCP];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (k + u < nsplit)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            sx[i] += split_sign(u) * v[u][i].x;
            sy[i] += split_sign(u) * v[u][i].y;
          }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (t0 + i < T) {
        sx[i] *= inv_z;
        sy[i] *= inv_z;
        if (y_meas) {
          sx[i] -= m[i].x;
          sy[i] -= m[i].y;
        }
        y[i] = make_float2((float)sx[i], (float)sy[i]);
      }
    // (padded samples stay zero)
  }
  const float sc = data_scale(bnd, nbnd, src ? 0 : nsplit, inv_z, bnd_meas, (int)pz);
  if (blockIdx.x == 0 && threadIdx.x == 0) scl[2 * pz + 1] = sc;
  if (!live) return;
  const float f = sc * split_sign(16 * (qg / NGP) / chunk);
  if (yop && !im) {
#pragma unroll
    for (int i = 0; i < 8; ++i) yop[(pz * Tp + t0 + i) * NCP + col] = y[i];
  }
  float b1[8], b2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    b1[i] = (im ? y[i].y : y[i].x) * f;
    b2[i] = (im ? -y[i].x : y[i].y) * f;
  }
  write_rec3(ys + (pz * (Tp / 16) * NGP + qg) * kRec3 + lane, b1, b2);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

// Reduction splits and column blocks of a forward launch.
struct Pass {
  int split0, nsplit, gy0, ngy;
};
static Pass whole(const EncPlan &p) { return Pass{0, p.fwd_split, 0, p.NGY}; }
static int pass_pixels(const EncPlan &p, const Pass &w) {
  return (int)std::min<int64_t>(p.Rp - (int64_t)w.split0 * p.fwd_chunk, (int64_t)w.nsplit * p.fwd_chunk);
}

// go(column groups per wave, FOLD)
template <class Go>
static void variant(const EncPlan &p, bool fold, Go go) {
  using One = std::integral_constant<int, 1>;
  using Two = std::integral_constant<int, 2>;
  if (fold) p.GW == 2 ? go(Two{}, std::true_type{}) : go(One{}, std::true_type{});
  else p.GW == 2 ? go(Two{}, std::false_type{}) : go(One{}, std::false_type{});
}

template <int NT>
static void launch_forward(const EncPlan &p, const EncBuffers &b, const Pass &w, hipStream_t s) {
  const int pix0 = w.split0 * p.fwd_chunk;
  const double *own = NT ? b.kap : b.pmono, *uni = NT ? b.bet + (size_t)pix0 * NT : b.dwq + pix0;
  const u32x4 *op = reinterpret_cast<const u32x4 *>(b.zs);
  float *part = reinterpret_cast<float *>(b.part + ((int64_t)w.split0 * p.Tp * p.NCP + w.gy0 * p.GW * 16));
  const F32Args a{p.Tp, pass_pixels(p, w), p.NCP, w.ngy * p.GW, p.fwd_chunk, w.nsplit, p.nxq, p.nx, p.ny, pix0,
                  p.dx, p.dy, bf16_masks(), b.wmax};
  const dim3 grid(split_grid(p.Tp / 256 * w.nsplit), (unsigned)w.ngy, (unsigned)p.P);
  variant(p, p.fwd_fold, [&](auto gw, auto fold) {
    k_fwd_f32<NT, decltype(gw)::value, decltype(fold)::value><<<grid, 256, 0, s>>>(own, uni, op, part, a);
  });
}

// Image rows that a workgroup's 256 pixels can touch.  Workgroups start at
// multiples of 256, so in a row at multiples of gcd(256, nxq).
constexpr int kMaxRows = 16;  // nxq is a multiple of 16
static int block_rows(const EncPlan &p) {
  return (int)std::min<int64_t>((p.nxq - std::gcd(256, p.nxq) + 255) / p.nxq + 1, ceil_div(p.Rp, p.nxq));
}
static size_t adj_sh_lds(int nrow) { return (size_t)2 * kSamples * (4 * nrow + 1) * sizeof(double); }

template <int NT>
static int launch_adjoint(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  int st = EXPENC_OK;
  const u32x4 *op = reinterpret_cast<const u32x4 *>(b.ys);
  float *part = reinterpret_cast<float *>(b.part);
  const F32Args a{p.Tp, p.Rp, p.NCP, p.NCP / 16, p.adj_chunk, p.adj_split, p.nxq, p.nx, p.ny, 0,
                  p.dx, p.dy, bf16_masks(), nullptr};
  const dim3 grid(split_grid((int64_t)p.Rp / 256 * p.adj_split), (unsigned)p.NGY, (unsigned)p.P);
  variant(p, p.adj_fold, [&](auto gw, auto fold) {
    constexpr int GW = decltype(gw)::value;
    constexpr bool FOLD = decltype(fold)::value;
    if constexpr (NT > 0) {
      k_adj_f32<NT, GW, FOLD><<<grid, 256, 0, s>>>(b.bet, b.kap, op, part, a);
    } else {
      const int nrow = block_rows(p);
      st = allow_lds(reinterpret_cast<const void *>(k_adj_f32_sh<GW, FOLD>), adj_sh_lds(nrow), adj_sh_lds(kMaxRows));
      if (st == EXPENC_OK)
        k_adj_f32_sh<GW, FOLD><<<grid, 256, adj_sh_lds(nrow), s>>>(b.pmono, b.dwq, op, part, a, nrow);
    }
  });
  return st;
}

static void forward_pass(const EncPlan &p, const EncBuffers &b, const Pass &w, hipStream_t s) {
  if (p.sh) return launch_forward<0>(p, b, w, s);
  switch (p.NT) {
    case 4: return launch_forward<4>(p, b, w, s);
    case 10: return launch_forward<10>(p, b, w, s);
    default: return launch_forward<17>(p, b, w, s);
  }
}

void f32_forward_launch(const EncPlan &p, const EncBuffers &b, hipStream_t s) { forward_pass(p, b, whole(p), s); }

int f32_adjoint_launch(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  if (p.sh) return launch_adjoint<0>(p, b, s);
  switch (p.NT) {
    case 4: return launch_adjoint<4>(p, b, s);
    case 10: return launch_adjoint<10>(p, b, s);
    default: return launch_adjoint<17>(p, b, s);
  }
}

static dim3 record_grid(int64_t len, int groups, const EncPlan &p) {
  return dim3((unsigned)ceil_div(len / 16 * groups * 64, 256), (unsigned)p.P);
}

// the records of a pass, of an image that is bounded
static int build_z(const EncPlan &p, const float *smaps, const float2 *x, int64_t x_stride, int32_t x_row_stride,
                   const EncBuffers &b, const Pass &w, hipStream_t s, int64_t x_pstride) {
  const int npix = pass_pixels(p, w), groups = w.ngy * p.GW;
  k_build_z_f32<<<record_grid(npix, groups, p), 256, 0, s>>>(
      reinterpret_cast<const float2 *>(smaps), x, x_stride, x_row_stride, p.nx, p.ny, p.nxq, npix,
      w.split0 * p.fwd_chunk, p.C, p.NC, w.gy0 * p.GW, groups, reinterpret_cast<u32x4 *>(b.zs), x_pstride,
      p.fwd_chunk, b.amax, b.scl);
  EX_LAUNCHED("build_z");
  return EXPENC_OK;
}

int f32_build_z(const EncPlan &p, const float *smaps, const float2 *x, int64_t x_stride, int32_t x_row_stride,
                const EncBuffers &b, hipStream_t s, int64_t x_pstride, bool prepared) {
  if (!prepared) EX_TRY(bound_image(p, x, nullptr, x_stride, x_row_stride, x_pstride, b, s));
  return build_z(p, smaps, x, x_stride, x_row_stride, b, whole(p), s, x_pstride);
}

int f32_forward_passes(const EncPlan &p, const float *smaps, const float2 *x, const EncBuffers &b, hipStream_t s) {
  for (int s0 = 0; s0 < p.fwd_split; s0 += p.pass_split)
    for (int g0 = 0; g0 < p.NGY; g0 += p.pass_gy) {
      const Pass w{s0, std::min(p.pass_split, p.fwd_split - s0), g0, std::min(p.pass_gy, p.NGY - g0)};
      EX_TRY(build_z(p, smaps, x, p.R, p.nx, b, w, s, 0));
      forward_pass(p, b, w, s);
      EX_LAUNCHED("forward contraction");
    }
  return EXPENC_OK;
}

int f32_pack_y(const EncPlan &p, const float2 *y, float sign, const float2 *y_meas, const EncBuffers &b,
               hipStream_t s, bool prepared, bool *y_bounded) {
  DataBound d;
  EX_TRY(bound_data(p, y, y_meas, b, prepared, y_bounded, &d, s));
  k_pack_y_f32<<<record_grid(p.Tp, p.NCP / 16, p), 256, 0, s>>>(
      y, sign, p.adj_chunk, b.part, p.fwd_split, y_meas, p.T, p.Tp, p.C, p.NC, p.NCP,
      reinterpret_cast<u32x4 *>(b.ys), y ? nullptr : b.yop, d.bnd, d.nbnd, d.meas, b.scl);
  EX_LAUNCHED("pack_y");
  return EXPENC_OK;
}

}  // namespace expenc
