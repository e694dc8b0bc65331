// Split-precision (bf16 or fp16 hi+lo) forms of the encoding contractions.
//
// Every operand value v (FP32) is written as hi + lo with hi = rnd(v) and
// lo = rnd(v - hi) in the 16-bit format; a product a*b is taken as
// a_hi*b_hi + a_hi*b_lo + a_lo*b_hi on v_mfma_f32_32x32x16_{bf16,f16} with FP32
// accumulation (the lo*lo term, ~2^-2p relative, is dropped).  This runs the
// contraction at the 16-bit MFMA rate with an error of about 3*2^-16 per
// product (bf16) or 3*2^-22 (fp16) instead of 2^-8 / 2^-11 for a plain
// 16-bit product.
//
// Layout of one MFMA step (K = 16 reduction indices): lane l holds 8
// reduction indices, in the polynomial forward the consecutive ones 8*(l/32) .. 8*(l/32)+7 of row l%32 for the A
// operand and of column l%32 for the B operand.  In the polynomial forward, as
// in the FP32 kernels, each lane first evaluates the phases of ITS OWN row at all 16
// reduction indices (which are wave-uniform, so their field/basis values
// come through scalar loads), splits and packs pairs into 32-bit words, and
// v_permlane32_swap exchanges the half-waves so that the two 32-row MFMA
// blocks receive their operands (the other kernels take their phases from a
// matrix product in that layout).  The B operand is pre-split and packed in
// exactly the per-lane order (four 16-byte records per lane and step: b1 hi,
// b1 lo, b2 hi, b2 lo), so the inner loop loads it with dwordx4 loads.
#include <algorithm>
#include <vector>

#include "internal.h"
#include "split_dev.h"

namespace expenc {

// Slot of this wave in the per-problem maxima array of a forward launch
// (workgroup bx, by of a grid gx wide).
__device__ inline int wave_slot(int bx, int by, int gx) { return (by * gx + bx) * 4 + (threadIdx.x >> 6); }

// ---------------------------------------------------------------------------
// Split forms with the solid-harmonic basis in polynomial form.  With z
// fixed, sum_l k_l(t) b_l(x, y) is a cubic polynomial in (x, y) whose ten
// monomial coefficients P_m(t) (turns) are formed once per sample.
//
// Forward (lane = sample t, 16 pixels of one image row per step): along the
// row the phase is a cubic in x.  Each lane expands it around the tile
// centre x_c in FP64: the anchor phi(x_c) reduced to [0,1), and the scaled
// Taylor coefficients d1 = phi_x dx, d2 = phi_xx dx^2 / 2, d3 = phi_xxx dx^3 / 6.
// Pixel x_c + k dx (k = -8..7, a literal) then costs three FP32 FMAs, plus
// one for the off-resonance difference t (dw0(r) - dw0(r_c)) / 2pi.
//
// Adjoint (32 samples x 64 pixels per wave and step): the phase is the
// FP64 anchor of the tile's centre sample t_c at each pixel (a table written
// at preparation) plus the increment sum_m (P_m(t) - P_m(t_c)) mono_m(r) +
// (t - t_c) dw0(r)/2pi.  Inside one image row the increment is a cubic in x
// whose four coefficients are polynomials in the row's y, so for a block of
// 32 pixels of one row it is a rank-6 product (the cubic, dw0 and the
// anchor with a unit A entry) of a [32 samples x 6] operand, evaluated per
// block from per-sample coefficients, with a [6 x 32 pixels] operand: three
// v_mfma_f32_32x32x2_f32 per block (five for a block that continues into
// the next row), instead of eleven FP32 FMAs per entry on the vector unit.
// The product's output layout gives each lane 16 samples of ONE
// pixel, which is the A-operand layout of the contraction up to a fixed
// permutation of the samples inside each group of 16; the adjoint records
// are packed in that order, so no exchange between lanes is needed.
// ---------------------------------------------------------------------------

// Arguments of one problem group's forward launch.
struct FwdShArgs {
  const double *pmono, *dwq;
  const float *ddw;
  const u32x4 *zs;
  float *part, *wmax;
  int64_t Tp;
  int Rp, NCP, chunk, nsplit, nxq, nx, ny;
  double dx, dy;
  Bf16Masks mk;
};

// One workgroup of the forward (workgroup bx, by, bz of a gx x gy x P grid).
template <int GW, bool BF, bool FOLD>
__device__ inline void fwd_split_sh_body(const FwdShArgs &a, int bx, int by, int bz, int gx, int gy) {
  const double *__restrict__ pmono = a.pmono;
  const double *__restrict__ dwq = a.dwq;
  const float *__restrict__ ddw = a.ddw;
  const u32x4 *__restrict__ zs = a.zs;
  float *__restrict__ part = a.part;
  float *__restrict__ wmax = a.wmax;
  const int64_t Tp = a.Tp;
  const int Rp = a.Rp, NCP = a.NCP, chunk = a.chunk, nsplit = a.nsplit, nxq = a.nxq, nx = a.nx, ny = a.ny;
  const double dx = a.dx, dy = a.dy;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int split, rb;
  if (wmax) wmax += (int64_t)bz * gy * gx * 4;
  const int slot = wave_slot(bx, by, gx);
  if (!split_tile(bx, (int)(Tp / 256), nsplit, &split, &rb)) {
    if (wmax && lane == 0) wmax[slot] = 0.f;
    return;
  }
  const int64_t row0 = (int64_t)rb * 256 + wave * 64;
  const int g0 = by * GW;
  const int NGP = NCP / 16;
  const int pz = bz;  // problem
  pmono += pz * Tp * kPolyStride;
  dwq += (int64_t)pz * Rp;
  ddw += (int64_t)pz * Rp;
  zs += (int64_t)pz * Rp * NGP * 16;
  part += pz * nsplit * Tp * NCP * 2;
  double P[10];
#pragma unroll
  for (int m = 0; m < 10; ++m) P[m] = pmono[(row0 + lane) * kPolyStride + m];
  const double tt = pmono[(row0 + lane) * kPolyStride + 10];
  const float tf = (float)tt;
  const double dx2 = dx * dx, dx3 = dx2 * dx;
  f32x16 acc[2][GW];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int g = 0; g < GW; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][g][v] = 0.f;
  const int r0 = split * chunk;
  const int r1 = min(Rp, r0 + chunk);
  // Software pipeline: the phases of tile r + 16 are evaluated between the
  // MFMAs of tile r, in ten slots of a few MFMAs and the vector work of two
  // indexes.  The vector unit issues in three quarters of the cycles and the
  // matrix cores are busy in half, at a clock of 1.9 GHz that the two share;
  // left to itself the compiler puts the MFMAs behind the phases, the more so
  // the fewer vector instructions those take: against the cubic expanded anew
  // for every tile, 148 x 148, 32 coils, T = 16384 (fp16) took 7 % more time with
  // it moved along the row, and takes 3 % less pipelined.
  u32x4 A[2][4], bq[GW][4];
  f32x16 ts[2];      // FOLD: a column group's sums over the tile
  uint32_t w[4][8];  // [kind: c hi, c lo, s hi, s lo][pair of indexes]
  float ph[16], dd[16];
  RowCubic rc;  // of the tile whose phases come next
  rc.start(r0, nxq);
  double dq = 0.0;
  auto load_b = [&](int g, int r) {
    const u32x4 *zq = zs + ((int64_t)(r >> 4) * NGP + (g0 + g)) * 256 + lane;
    bq[g][0] = zq[0];
    bq[g][1] = zq[64];
    bq[g][2] = zq[128];
    bq[g][3] = zq[192];
  };
  auto load_dw = [&](int r) {
    dq = dwq[r + 8];
#pragma unroll
    for (int j = 0; j < 16; ++j) dd[j] = ddw[r + j];
  };
  auto expand = [&] {
    rc.expand(P, nx, ny, dx, dy, dx2, dx3);
    rc.next(nxq);
    const float an = (float)__builtin_amdgcn_fract(fma(tt, dq, rc.c0));
    const float d1 = (float)rc.d1, d2 = (float)rc.d2, d3 = (float)rc.d3;
    // p(k) = an + d1 k + d2 k^2 + d3 k^3 at k = j - 8: the even part
    // an + d2 k^2 and the odd factor d1 + d3 k^2 are shared by k and -k
    ph[8] = an;
#pragma unroll
    for (int m = 1; m < 8; ++m) {
      const float k = (float)m, k2 = (float)(m * m);
      const float ev = fmaf(d2, k2, an), od = fmaf(d3, k2, d1);
      ph[8 + m] = fmaf(od, k, ev);
      ph[8 - m] = fmaf(od, -k, ev);
    }
    ph[0] = fmaf(fmaf(fmaf(d3, -8.f, d2), -8.f, d1), -8.f, an);
  };
  auto pair = [&](int m) {
    float c2[2], s2[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float f = __builtin_amdgcn_fractf(fmaf(tf, dd[2 * m + e], ph[2 * m + e]));
      c2[e] = __builtin_amdgcn_cosf(f);
      s2[e] = __builtin_amdgcn_sinf(f);
    }
    split_pair<BF>(c2[0], c2[1], w[0][m], w[1][m], a.mk);
    split_pair<BF>(s2[0], s2[1], w[2][m], w[3][m], a.mk);
  };
  auto exchange = [&] {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto x = __builtin_amdgcn_permlane32_swap(w[q][i], w[q][4 + i], false, false);
        A[0][q][i] = x[0];
        A[1][q][i] = x[1];
      }
  };
  // MFMAs [lo, hi) of a tile: column groups in turn, the products of the two
  // row blocks alternating
  auto products = [&](int lo, int hi) {
    constexpr int pa[6] = {0, 0, 1, 2, 2, 3}, pb[6] = {0, 1, 0, 2, 3, 2};
#pragma unroll
    for (int k = 0; k < 12 * GW; ++k)
      if (k >= lo && k < hi) {
        const int g = k / 12, q = k % 12 >> 1, blk = k & 1;
        f32x16 &c = FOLD ? ts[blk] : acc[blk][g];
        if (FOLD && k % 12 < 2) c = f32x16{};
        c = mfma16<BF>(A[blk][pa[q]], bq[g][pb[q]], c);
        if (FOLD && k % 12 >= 10) acc[blk][g] += c;
      }
  };
  load_dw(r0);
#pragma unroll
  for (int g = 0; g < GW; ++g) load_b(g, r0);
  expand();
#pragma unroll
  for (int m = 0; m < 8; ++m) pair(m);
  exchange();
  for (int r = r0; r + 16 < r1; r += 16) {
    constexpr int N = 12 * GW;
    load_dw(r + 16);
    products(0, N / 10);
    __builtin_amdgcn_sched_barrier(0);
    products(N / 10, N * 2 / 10);
    expand();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      products(N * (m + 2) / 10, N * (m + 3) / 10);
      pair(m);
      // a column group's records are replaced once its products are issued
#pragma unroll
      for (int g = 0; g < GW; ++g)
        if (N * (m + 2) / 10 < 12 * (g + 1) && N * (m + 3) / 10 >= 12 * (g + 1)) load_b(g, r + 16);
    }
    exchange();
  }
  products(0, 12 * GW);
  store_partials<GW>(part + (int64_t)split * Tp * NCP * 2, row0, NCP, g0, lane, acc, wmax, slot);
}

// Waves per SIMD as without folds (three with 16 columns, two with 32): left to
// itself the compiler gives the folded kernels more registers than that allows.
// Held to it the one of 16 columns spills 18, and is the faster all the same:
// 46 us for 50 at 100 x 90, 16 coils, T 3000 (fp16), 82 for 88 with 4 images.
template <int GW, bool BF, bool FOLD>
__global__ __launch_bounds__(256, 4 - GW) void k_fwd_split_sh(FwdShArgs a) {
  fwd_split_sh_body<GW, BF, FOLD>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x, gridDim.y);
}

// One launch for several problem groups of one shape class (same GW and
// number format): the workgroups of every group's grid are numbered group by
// group (x fastest) and the launch has one workgroup per tile.  Every group's
// x extent is a multiple of eight, so a tile runs on the XCD its index
// assigns it and split_tile's L2 locality holds.  (A persistent form, a
// grid of the resident workgroups walking the tiles with its stride, was
// slower: its loop raised the adjoint's registers to two waves per SIMD.)
template <int GW, bool BF, bool FOLD>
__global__ __launch_bounds__(256, 4 - GW) void k_fwd_split_sh_grouped(GroupedLaunch<FwdShArgs> G) {
  {
    const int64_t t = blockIdx.x;
    if (t >= G.off[G.ng]) return;
    int g = 0;
    while (g + 1 < G.ng && t >= G.off[g + 1]) ++g;
    const int64_t l = t - G.off[g];
    const int gx = G.gx[g], gy = G.gy[g];
    const int64_t q = l / gx;
    fwd_split_sh_body<GW, BF, FOLD>(G.a[g], (int)(l - q * gx), (int)(q % gy), (int)(q / gy), gx, gy);
  }
}

// ---------------------------------------------------------------------------
// Operand packing.  Record (step q, group g, lane l): 8 reduction indices
// 16q + 8*(l/32) + i, column col = 16g + l%16, part = (l/16)&1.
//   forward:  b1 = part ? Zi : Zr,   b2 = part ? Zr : -Zi
//   adjoint:  b1 = part ? Yi : Yr,   b2 = part ? -Yr : Yi
// times the operand's scale and the sign of the index's split.  The adjoints and
// the general-basis forward read the indices of a step in the order of k_pack_y_split.
// ---------------------------------------------------------------------------

// Max of m over workgroup blk of nblk into its slots blk, blk + nblk, ... of
// the kAmaxBlocks in out.
__device__ inline void write_block_max(float m, float *__restrict__ out, int blk, int nblk) {
  __shared__ float wm[4];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  const int slot = blk + threadIdx.x * nblk;
  if (slot < kAmaxBlocks) out[slot] = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
}

// Pre-pass of the image operand: per-workgroup max of |Re u| + |Im u| over
// the encoded pixels and images, u = x - xsub.  With the same bound of the
// coil maps (taken once per preparation), their product bounds the
// components of Z = S u.  Grid (at most kAmaxBlocks, P), 256 threads.
__global__ __launch_bounds__(256) void k_amax_z(const float2 *__restrict__ x, const float2 *__restrict__ xsub,
                                                int64_t x_stride, int x_row_stride, int nx, int ny, int B,
                                                int64_t x_pstride, float *__restrict__ amax) {
  const int pz = blockIdx.y;
  const int R = nx * ny;
  x += pz * x_pstride;
  if (xsub) xsub += pz * x_pstride;
  float m = 0.f;
  for (int r = blockIdx.x * 256 + threadIdx.x; r < R; r += gridDim.x * 256) {
    const int yy = r / nx, xx = r % nx;
    for (int b = 0; b < B; ++b) {
      const int64_t o = b * x_stride + (int64_t)yy * x_row_stride + xx;
      float2 u = x[o];
      if (xsub) {
        u.x -= xsub[o].x;
        u.y -= xsub[o].y;
      }
      m = fmaxf(m, magnitude(u, true));
    }
  }
  write_block_max(m, amax + pz * kAmaxBlocks, blockIdx.x, gridDim.x);
}

// Pre-pass of a complex array [P][n] (stride pstride): per-workgroup max of
// the component magnitudes.  Grid (at most kAmaxBlocks, P), 256 threads.
__global__ __launch_bounds__(256) void k_amax_c(const float2 *__restrict__ v, int64_t n, int64_t pstride,
                                                float *__restrict__ amax) {
  const int pz = blockIdx.y;
  v += pz * pstride;
  float m = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    m = fmaxf(m, magnitude(v[i], false));
  }
  write_block_max(m, amax + pz * kAmaxBlocks, blockIdx.x, gridDim.x);
}

// (perm: the index order of the adjoint records below, which the
// general-basis forward shares)
template <bool BF>
__global__ __launch_bounds__(256) void k_build_z_split(const float2 *__restrict__ smaps, const float2 *__restrict__ x,
                                const float2 *__restrict__ xsub, int64_t x_stride, int x_row_stride, int nx, int ny,
                                int nxq, int Rp, int C, int NC, int NGP, u32x4 *__restrict__ zs, int64_t x_pstride,
                                const float2 *__restrict__ sq, const float *__restrict__ amax,
                                float *__restrict__ scl, int perm, int chunk) {
  const int R = nx * ny;
  const int pz = blockIdx.y;  // problem
  // scaled form: every workgroup derives the same power of two from the pre-pass
  float sc = 1.f;
  if (scl) {
    sc = image_scale(amax, pz, gridDim.y);
    if (blockIdx.x == 0 && threadIdx.x == 0) scl[2 * pz] = sc;
  }
  smaps += (int64_t)pz * C * R;
  if (sq) sq += (int64_t)pz * Rp * NGP * 16;
  x += pz * x_pstride;
  if (xsub) xsub += pz * x_pstride;
  zs += (int64_t)pz * Rp * NGP * 16;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)(Rp / 16) * NGP * 64) return;
  const int lane = (int)(id & 63);
  const int g = (int)((id >> 6) % NGP);
  const int64_t q = (id >> 6) / NGP;
  const int col = 16 * g + (lane & 15);
  const int im = (lane >> 4) & 1;
  // the 8 pixels of this lane: every load is issued before the arithmetic
  // (outside pixels and columns read an in-bounds element and give 0)
  const int half = lane >> 5, rq0 = (int)(16 * q) + (perm ? 4 : 8) * half;
  int rq = rq0, yy = rq / nxq, xx = rq - yy * nxq;
  const bool colok = col < NC;
  const int b = colok ? col / C : 0, c = colok ? col % C : 0;
  float2 u[8], w[8], sv[8];
  bool ok[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    ok[i] = yy < ny && xx < nx && colok;
    const int yc = ok[i] ? yy : 0, xc = ok[i] ? xx : 0;
    const int64_t o = b * x_stride + (int64_t)yc * x_row_stride + xc;
    u[i] = x[o];
    w[i] = xsub ? xsub[o] : make_float2(0.f, 0.f);
    // (the S table, when given, holds the same value in row-major order)
    sv[i] = sq ? sq[(int64_t)rq * NGP * 16 + col] : smaps[(int64_t)c * R + yc * nx + xc];
    const int step = perm && i == 3 ? 5 : 1;
    rq += step;
    xx += step;
    while (xx >= nxq) {
      xx -= nxq;
      ++yy;
    }
  }
  const float f = sc * split_sign(16 * q / chunk);
  float b1[8], b2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float2 uu = u[i];
    if (xsub) {
      uu.x -= w[i].x;
      uu.y -= w[i].y;
    }
    const float2 s = sv[i];
    const float2 z = ok[i] ? make_float2((s.x * uu.x - s.y * uu.y) * f, (s.x * uu.y + s.y * uu.x) * f)
                           : make_float2(0.f, 0.f);
    b1[i] = im ? z.y : z.x;
    b2[i] = im ? z.x : -z.y;
  }
  write_record<BF>(zs, q, g, NGP, lane, b1, b2);
}

// Adjoint operand from y [B][T][C] (src_abi) or from forward partials minus
// y_meas (src_part, nsplit partial arrays in [Tp][NCP] layout).
// K index 8h + i of a step holds sample 8(i/4) + 4h + i%4 of its 16 (the
// order in which the adjoints produce their phase tiles).
template <bool BF>
__global__ __launch_bounds__(256) void k_pack_y_split(const float2 *__restrict__ src_abi,
                                                      const float2 *__restrict__ src_part, int nsplit,
                                                      const float2 *__restrict__ y_meas, int64_t T, int64_t Tp, int C,
                                                      int NC, int NCP, u32x4 *__restrict__ ys,
                                                      const float *__restrict__ bnd, int nbnd,
                                                      const float *__restrict__ bnd_meas, float *__restrict__ scl,
                                                      int chunk) {
  const int NGP = NCP / 16;
  const int pz = blockIdx.y;  // problem
  float sc = 1.f, inv_z = 1.f;
  if (scl) {
    if (src_part) inv_z = 1.f / scl[2 * pz];
    sc = data_scale(bnd, nbnd, src_part ? nsplit : 0, inv_z, bnd_meas, pz);
    if (blockIdx.x == 0 && threadIdx.x == 0) scl[2 * pz + 1] = sc;
  }
  if (src_abi) src_abi += pz * T * NC;
  if (src_part) src_part += pz * nsplit * Tp * NCP;
  if (y_meas) y_meas += pz * T * NC;
  ys += pz * Tp * NGP * 16;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (Tp / 16) * NGP * 64) return;
  const int lane = (int)(id & 63);
  const int g = (int)((id >> 6) % NGP);
  const int64_t q = (id >> 6) / NGP;
  const int col = 16 * g + (lane & 15);
  const int im = (lane >> 4) & 1;
  const int b = col / C, c = col % C;
  int64_t t[8];
  bool ok[8];
  float2 y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    t[i] = 16 * q + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
    ok[i] = t[i] < T && col < NC;
    y[i] = make_float2(0.f, 0.f);
  }
  if (src_abi) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (ok[i]) y[i] = src_abi[((int64_t)b * T + t[i]) * C + c];
  } else {
    // split order per sample as in a plain loop; the loads of four splits x
    // eight samples are independent and issue together (unconditional, padded
    // rows and columns exist: under a branch the compiler puts the sign's
    // negation, and with it a wait, after every load)
    int k = 0;
    for (; k + 4 <= nsplit; k += 4) {
      float2 v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          v[u][i] = src_part[((int64_t)(k + u) * Tp + t[i]) * NCP + col];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          y[i].x += split_sign(u) * v[u][i].x;
          y[i].y += split_sign(u) * v[u][i].y;
        }
    }
    if (k < nsplit) {  // the last splits repeated
      float2 v[3][8];
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          v[u][i] = src_part[((int64_t)min(k + u, nsplit - 1) * Tp + t[i]) * NCP + col];
#pragma unroll
      for (int u = 0; u < 3; ++u)
        if (k + u < nsplit)
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            y[i].x += split_sign(u) * v[u][i].x;
            y[i].y += split_sign(u) * v[u][i].y;
          }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      y[i].x = ok[i] ? y[i].x * inv_z : 0.f;
      y[i].y = ok[i] ? y[i].y * inv_z : 0.f;
    }
    if (y_meas) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (ok[i]) {
          const float2 m = y_meas[((int64_t)b * T + t[i]) * C + c];
          y[i].x -= m.x;
          y[i].y -= m.y;
        }
    }
  }
  const float f = sc * split_sign(16 * q / chunk);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    y[i].x *= f;
    y[i].y *= f;
  }
  float b1[8], b2[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    b1[i] = im ? y[i].y : y[i].x;
    b2[i] = im ? -y[i].x : y[i].y;
  }
  write_record<BF>(ys, q, g, NGP, lane, b1, b2);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

static FwdShArgs fwd_sh_args(const EncPlan &p, const EncBuffers &b) {
  return FwdShArgs{b.pmono, b.dwq, b.ddw, reinterpret_cast<const u32x4 *>(b.zs), reinterpret_cast<float *>(b.part),
                   p.scaled ? b.wmax : nullptr, p.Tp, p.Rp, p.NCP, p.fwd_chunk, p.fwd_split, p.nxq, p.nx, p.ny,
                   p.dx, p.dy, bf16_masks()};
}

static void fwd_split_sh(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  dim3 grid(split_grid(p.Tp / 256 * p.fwd_split), (unsigned)p.NGY, (unsigned)p.P);
  const FwdShArgs a = fwd_sh_args(p, b);
  split_variant(p, p.fwd_fold, [&](auto gw, auto bf, auto fold) {
    k_fwd_split_sh<gw.value, bf.value, fold.value><<<grid, 256, 0, s>>>(a);
  });
}

bool split_groupable(const EncPlan &a, const EncPlan &b) {
  return a.sh && b.sh && a.prec == b.prec && a.prec != EXPENC_FP32 && a.GW == b.GW && a.comb == b.comb &&
         a.scaled == b.scaled;
}

static int fwd_grouped(const EncPlan *const *p, const EncBuffers *const *b, int n, hipStream_t s) {
  GroupedLaunch<FwdShArgs> G{};
  G.ng = n;
  G.off[0] = 0;
  for (int g = 0; g < n; ++g) {
    G.a[g] = fwd_sh_args(*p[g], *b[g]);
    G.gx[g] = (int)split_grid(p[g]->Tp / 256 * p[g]->fwd_split);
    G.gy[g] = p[g]->NGY;
    G.off[g + 1] = G.off[g] + (int64_t)G.gx[g] * G.gy[g] * p[g]->P;
  }
  if (G.off[n] > INT32_MAX) return fail(EXPENC_EUNSUPPORTED, "grouped launch larger than 2^31 workgroups");
  split_variant(*p[0], p[0]->fwd_fold, [&](auto gw, auto bf, auto fold) {
    k_fwd_split_sh_grouped<gw.value, bf.value, fold.value><<<(unsigned)G.off[n], 256, 0, s>>>(G);
  });
  EX_LAUNCHED("grouped forward contraction");
  return EXPENC_OK;
}

int split_forward_grouped(const EncPlan *const *p, const EncBuffers *const *b, int n, hipStream_t s) {
  // (groups of folded sums and the others take kernels of their own)
  std::vector<const EncPlan *> pv[2];
  std::vector<const EncBuffers *> bv[2];
  for (int g = 0; g < n; ++g) {
    if (!split_groupable(*p[0], *p[g])) return fail(EXPENC_EINVAL, "plans of a grouped launch differ in shape");
    pv[p[g]->fwd_fold].push_back(p[g]);
    bv[p[g]->fwd_fold].push_back(b[g]);
  }
  for (int f = 0; f < 2; ++f)
    for (int i = 0; i < (int)pv[f].size(); i += kMaxGrouped)
      EX_TRY(fwd_grouped(pv[f].data() + i, bv[f].data() + i, std::min(kMaxGrouped, (int)pv[f].size() - i), s));
  return EXPENC_OK;
}

void split_forward_launch(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  if (p.sh) fwd_split_sh(p, b, s);
  else split_maps_launch(p, b, false, s);
}

void split_adjoint_launch(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  if (p.sh) split_adjoint_sh_launch(p, b, s);
  else split_maps_launch(p, b, true, s);
}

int bound_image(const EncPlan &p, const float2 *x, const float2 *xsub, int64_t x_stride, int32_t x_row_stride,
                int64_t x_pstride, const EncBuffers &b, hipStream_t s) {
  if (!b.scl || !b.amax || !b.wmax) return fail(EXPENC_EINVAL, "scale buffers of a scaled plan are not carved");
  k_amax_z<<<dim3(amax_blocks((int64_t)p.R * p.B), (unsigned)p.P), 256, 0, s>>>(x, xsub, x_stride, x_row_stride, p.nx, p.ny, p.B,
                                                            x_pstride, b.amax);
  EX_LAUNCHED("operand bound");
  return EXPENC_OK;
}

int bound_data(const EncPlan &p, const float2 *y, const float2 *y_meas, const EncBuffers &b, bool prepared,
               bool *y_bounded, DataBound *d, hipStream_t s) {
  if (!b.scl || !b.amax || !b.wmax) return fail(EXPENC_EINVAL, "scale buffers of a scaled plan are not carved");
  auto pass = [&](const float2 *v, int64_t n, float *out) -> int {
    k_amax_c<<<dim3(amax_blocks(n), (unsigned)p.P), 256, 0, s>>>(v, n, n, out);
    EX_LAUNCHED("operand bound");
    return EXPENC_OK;
  };
  const int64_t ny_el = p.T * p.NC;  // [B][T][C] per problem
  d->bnd = b.amax;
  d->nbnd = kAmaxBlocks;
  if (y) return prepared ? EXPENC_OK : pass(y, ny_el, b.amax);
  if (p.sh || p.prec == EXPENC_FP32) {
    // these forwards write their per-wave output maxima
    d->bnd = b.wmax;
    d->nbnd = p.nwmax;
  } else {
    // (the split maps-kind forward does not: a pre-pass over its partial sums)
    EX_TRY(pass(b.part, (int64_t)p.fwd_split * p.Tp * p.NCP, b.amax));
  }
  if (y_meas) {
    float *am = b.amax + (size_t)p.P * kAmaxBlocks;
    if (!y_bounded || !*y_bounded) EX_TRY(pass(y_meas, ny_el, am));
    if (y_bounded) *y_bounded = true;
    d->meas = am;
  }
  return EXPENC_OK;
}

int split_build_z(const EncPlan &p, const float *smaps, const float2 *x, const float2 *xsub, int64_t x_stride,
                  int32_t x_row_stride, const EncBuffers &b, hipStream_t s, int64_t x_pstride, bool prepared) {
  const int NGP = p.NCP / 16;
  const int64_t n = (int64_t)(p.Rp / 16) * NGP * 64;
  const dim3 nb((unsigned)ceil_div(n, 256), (unsigned)p.P);
  const float2 *sm = reinterpret_cast<const float2 *>(smaps);
  u32x4 *zs = reinterpret_cast<u32x4 *>(b.zs);
  if (p.scaled && !prepared) EX_TRY(bound_image(p, x, xsub, x_stride, x_row_stride, x_pstride, b, s));
  float *scl = p.scaled ? b.scl : nullptr;
  const float2 *sq = p.comb && !prepared ? b.sq : nullptr;
  if (p.prec == EXPENC_BF16_SPLIT)
    k_build_z_split<true><<<nb, 256, 0, s>>>(sm, x, xsub, x_stride, x_row_stride, p.nx, p.ny, p.nxq, p.Rp, p.C,
                                             p.NC, NGP, zs, x_pstride, sq, b.amax, scl, p.sh ? 0 : 1, p.fwd_chunk);
  else
    k_build_z_split<false><<<nb, 256, 0, s>>>(sm, x, xsub, x_stride, x_row_stride, p.nx, p.ny, p.nxq, p.Rp, p.C,
                                              p.NC, NGP, zs, x_pstride, sq, b.amax, scl, p.sh ? 0 : 1, p.fwd_chunk);
  EX_LAUNCHED("build_z split");
  return EXPENC_OK;
}

int split_pack_y(const EncPlan &p, const float2 *y_abi, bool from_partials, const float2 *y_meas,
                 const EncBuffers &b, hipStream_t s, bool prepared, bool *y_bounded) {
  const int NGP = p.NCP / 16;
  const int64_t n = (p.Tp / 16) * NGP * 64;
  const dim3 nb((unsigned)ceil_div(n, 256), (unsigned)p.P);
  u32x4 *ys = reinterpret_cast<u32x4 *>(b.ys);
  const float2 *part = from_partials ? b.part : nullptr;
  DataBound d;
  if (p.scaled) EX_TRY(bound_data(p, y_abi, y_meas, b, prepared, y_bounded, &d, s));
  float *scl = p.scaled ? b.scl : nullptr;
  if (p.prec == EXPENC_BF16_SPLIT)
    k_pack_y_split<true><<<nb, 256, 0, s>>>(y_abi, part, p.fwd_split, y_meas, p.T, p.Tp, p.C, p.NC, p.NCP, ys,
                                            d.bnd, d.nbnd, d.meas, scl, p.adj_chunk);
  else
    k_pack_y_split<false><<<nb, 256, 0, s>>>(y_abi, part, p.fwd_split, y_meas, p.T, p.Tp, p.C, p.NC, p.NCP, ys,
                                             d.bnd, d.nbnd, d.meas, scl, p.adj_chunk);
  EX_LAUNCHED("pack_y split");
  return EXPENC_OK;
}

}  // namespace expenc
