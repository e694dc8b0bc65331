// Gradients of the encoding operators with respect to the field parameters
// k_l(t) and dw0(r) (the differentiable form of eq. 1's operator).
//
// With E(t,r) = exp(i phi), phi = sum_l k_l(t) b_l(r) + dw0(r) t, one has
// dA/dk_l(t) = i b_l(r) A and dA/d dw0(r) = i t A.  For a real loss with
// upstream gradients in the convention grad = dL/dRe + i dL/dIm:
//   y = A x,    upstream g:   grad_k[t,l]  = -Im sum_c conj(g[t,c]) [A(b_l x)](t,c)
//                             grad_dw[r]   = -Im( x(r) conj([A^H (t g)](r)) )
//   x = A^H y,  upstream gx:  grad_k[t,l]  = -Im sum_c conj(y[t,c]) [A(b_l gx)](t,c)
//                             grad_dw[r]   = -Im( gx(r) conj([A^H (t y)](r)) )
// i.e. one form with (w, kk) = (x, g) or (gx, y).  Exchanging the sums over
// coils and pixels, both gradients are weighted sums of one real matrix,
//   V(t,r) = Im( E(t,r) M(t,r) ),  M(t,r) = sum_c conj(kk[t,c]) S_c(r) w(r),
//   grad_k[t,l] = -sum_r b_l(r) V(t,r),   grad_dw[r] = -sum_t t V(t,r),
// which is formed on the fly and never stored.  Per entry that is 4 C real
// products for M, one phase and L + 1 products, against 4 L C + 4 C and two
// phases for L basis-weighted forward products and an adjoint.
#include <algorithm>

#include "internal.h"
#include "reduce.h"
#include "split_dev.h"

namespace expenc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kGradChunkMax = 1024;  // pixels one workgroup accumulates in FP32
constexpr int kGradAmax = 64;        // workgroups of the magnitude pre-pass per array

// Per-workgroup max component magnitude of w [R] (blockIdx.y 0), kk [T][C] (1)
// and smaps [C][R] (2) into amax[3][kGradAmax].
__global__ __launch_bounds__(256) void k_grad_amax(const float2 *__restrict__ w, int64_t R,
                                                   const float2 *__restrict__ kk, int64_t T,
                                                   const float2 *__restrict__ smaps, int C,
                                                   float *__restrict__ amax) {
  __shared__ float wm[4];
  const float2 *v = blockIdx.y == 0 ? w : blockIdx.y == 1 ? kk : smaps;
  const int64_t m = blockIdx.y == 0 ? R : (blockIdx.y == 1 ? T : R) * C;
  float a = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m; i += (int64_t)gridDim.x * 256)
    a = fmaxf(a, fmaxf(fabsf(v[i].x), fabsf(v[i].y)));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a = fmaxf(a, __shfl_xor(a, o));
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) amax[blockIdx.y * gridDim.x + blockIdx.x] = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
}

// Power of two that brings the array's largest component into [1/2, 1) (1
// for an all-zero or non-finite array): M and the sums over it are FP32
// products of kk, w and the maps, and with all three scaled they are the same
// bits at any scale of the arrays.  The reductions divide the scales out in
// FP64.
__device__ inline float grad_scale(const float *__restrict__ amax) {
  float m = 0.f;
  for (int i = 0; i < kGradAmax; ++i) m = fmaxf(m, amax[i]);
  if (!(m > 0.f) || !(m <= 3.0e38f)) return 1.f;
  int e;
  (void)frexpf(m, &e);
  return ldexpf(1.f, min(126, max(-126, -e)));
}

// Operands of the gradient contraction, records of lane order.  za (rows:
// pixels, z_c = S_c w) and kb (columns: samples) hold, per block of 16 pixels
// or samples and group of 16 coils, three 16-byte words per lane (the exact
// bf16 parts hi, mid, lo): lane l has element l % 16 and, as reduction
// indices, real and imaginary part of coils 4 (l / 16) .. + 3.  tf[Tp] are the
// sample times; bt holds, per block of 16 pixels, b_{l % 16} at pixels
// 4 (l / 16) .. + 3 (from the table bet [Rp][NT], or the solid harmonics at
// the pixel centre).  Zero on padding.
struct GradPackArgs {
  const float2 *kk, *w, *smaps;
  const double *time, *bet;
  const float *amax;
  u32x4 *za, *kb;
  float *tf, *bt;
  int64_t T, Tp;
  int C, CK, NT, L, nx, ny, nxq, Rp;
  double dx, dy, z0;
};

__global__ __launch_bounds__(256) void k_grad_pack(GradPackArgs g) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nkb = g.Tp / 16 * g.CK * 64, nza = (int64_t)g.Rp / 16 * g.CK * 64;
  if (i < nkb + nza) {
    const bool samples = i < nkb;
    if (!samples) i -= nkb;
    const int lane = (int)i & 63, e = lane & 15;
    const int64_t rec = i >> 6, blk = rec / g.CK;
    const int c0 = (int)(rec % g.CK) * 16 + 4 * (lane >> 4);
    float2 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = make_float2(0.f, 0.f);
    if (samples) {
      const int64_t t = blk * 16 + e;
      if (t < g.T) {
        const float s = grad_scale(g.amax + kGradAmax);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (c0 + j < g.C) {
            const float2 k = g.kk[t * g.C + c0 + j];
            v[j] = make_float2(k.x * s, k.y * s);
          }
      }
    } else {
      const int r = (int)blk * 16 + e, yy = r / g.nxq, xx = r % g.nxq;
      if (xx < g.nx && yy < g.ny) {
        const float s = grad_scale(g.amax), sm = grad_scale(g.amax + 2 * kGradAmax);
        const int64_t pix = (int64_t)yy * g.nx + xx, R = (int64_t)g.nx * g.ny;
        float2 w = g.w[pix];
        w.x *= s;
        w.y *= s;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (c0 + j < g.C) {
            float2 c = g.smaps[(c0 + j) * R + pix];
            c.x *= sm;
            c.y *= sm;
            v[j] = make_float2(c.x * w.x - c.y * w.y, c.x * w.y + c.y * w.x);
          }
      }
    }
    u32x4 h, m, l;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t a, b, c;
      split3_any(v[j].x, v[j].y, a, b, c);
      h[j] = a;
      m[j] = b;
      l[j] = c;
    }
    u32x4 *o = (samples ? g.kb : g.za) + rec * 192 + lane;
    o[0] = h;
    o[64] = m;
    o[128] = l;
    return;
  }
  i -= nkb + nza;
  if (i < g.Tp) {
    g.tf[i] = i < g.T ? (float)g.time[i] : 0.f;
    return;
  }
  i -= g.Tp;
  if (i >= g.Rp) return;
  const int r = (int)i, yy = r / g.nxq, xx = r % g.nxq, e = r & 15;
  const bool in = xx < g.nx && yy < g.ny;
  double v[16];
  if (!g.bet) sh_eval((xx - 0.5 * g.nx) * g.dx, (yy - 0.5 * g.ny) * g.dy, g.z0, v);
  float *o = g.bt + (int64_t)(r >> 4) * 256 + 64 * (e >> 2) + (e & 3);
#pragma unroll
  for (int l = 0; l < 16; ++l) {
    float b = 0.f;
    if (in && l < g.L) b = (float)(g.bet ? g.bet[(int64_t)r * g.NT + min(l, g.NT - 1)] : v[l]);
    o[4 * l] = b;
  }
}

// Arguments of the gradient contraction.
struct GradArgs {
  float *gpart, *dpart;  // [nsplit][Tp][16], [Tp/256][Rp]; NULL: that gradient is not wanted
  int64_t Tp;
  int Rp, CK, ny, nx, nxq, chunk, nsplit;
  double dx, dy;
};

__device__ inline f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}

// sum over three exact parts each: the products below 2^-25 are left out
__device__ inline f32x4 mfma_3x3(const u32x4 (&a)[3], const u32x4 (&b)[3]) {
  f32x4 m = {0.f, 0.f, 0.f, 0.f};
  m = mfma_bf16(a[1], b[1], m);
  m = mfma_bf16(a[2], b[0], m);
  m = mfma_bf16(a[0], b[2], m);
  m = mfma_bf16(a[1], b[0], m);
  m = mfma_bf16(a[0], b[1], m);
  return mfma_bf16(a[0], b[0], m);
}

template <int CTRL>
__device__ inline float dpp(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xf, 0xf, false));
}

// One workgroup: 256 samples (64 per wave) x a chunk of pixels, in steps of
// 16 pixels, and 16 coils at a time (their sample operands stay in registers
// for the whole chunk).  Per step a wave forms M^T (rows: 16 pixels, columns:
// its samples in four blocks of 16) on v_mfma_f32_16x16x32_bf16 over the real
// and imaginary parts of 16 coils, from three exact bf16 parts per operand
// (6 products of 16 matrix cycles instead of 8 FP32 ones of 32); the second
// operand of Im M is the first with its halves exchanged.  Meanwhile each
// lane evaluates the FP64 phases of its own sample at the 16 wave-uniform
// pixels; two stages of lane exchanges bring them to M's layout.  V then sits
// with its sample in lane % 16 and its pixel 4 (lane / 16) + register, which
// is the A-operand layout of v_mfma_f32_16x16x4_f32, so grad_k is accumulated
// on the matrix cores without moving V.  That instruction adds its products one
// after the other, so a step's 16 pixels are summed from zero, in two halves, and
// join the chunk's sums in one addition.  Error of grad_k at the size below: 5.0e-7
// when they went through the accumulators, 1.7e-7 now, for 2.5 % of a training
// step's time (basis-weighted forwards, coils summed in FP64: 1.2e-6); 30 x 100, 5
// coils, 4 terms, T = 1000: 1.4e-7, 1.06e-7 (1.14e-7; 1.20e-7 without the halves).
// grad_dw sums over lanes by halving
// (DPP) into a row of LDS per wave: no barrier before the end of the chunk.
// The tables come as kernel parameters: only through those does the compiler
// read the wave-uniform ones by scalar loads.
// Bound: the matrix cores (768 cycles a step for M and 512 for the basis
// products) plus the vector work of 16 FP64 phases, sines and cosines, which
// does not overlap much with it.  At 128 x 128, 16 coils, T = 12000 and 16
// terms 0.26 ms; the same matrix on the FP32 instruction, its coil maps and
// data read again by every workgroup, took 0.68 ms, and the basis-weighted
// forward and adjoint before that 3.78 + 0.34 ms.
// NT 0: solid-harmonic kind (own: polynomial coefficients, uni: dwq); else
// the general basis (own: kap, uni: bet).
template <int NT>
__global__ __launch_bounds__(256, 2) void k_field_grad(const double *__restrict__ own, const double *__restrict__ uni,
                                                       const u32x4 *__restrict__ za, const u32x4 *__restrict__ kb,
                                                       const float *__restrict__ tf, const f32x4 *__restrict__ bt,
                                                       GradArgs a) {
  __shared__ float sdw[4][kGradChunkMax];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15;
  int split, rb;
  if (!split_tile(blockIdx.x, (int)(a.Tp / 256), a.nsplit, &split, &rb)) return;
  const int64_t t0 = (int64_t)rb * 256 + wave * 64;
  constexpr int NP = NT ? NT : 11;
  double P[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) P[j] = own[(t0 + lane) * (NT ? NT : kPolyStride) + j];
  float tm[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) tm[b] = tf[t0 + 16 * b + l16];
  const double dx2 = a.dx * a.dx, dx3 = dx2 * a.dx;
  f32x4 G[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) G[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int r0 = split * a.chunk, r1 = min(a.Rp, r0 + a.chunk);
  for (int ks = 0; ks < a.CK; ++ks) {
    u32x4 B[4][3];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int q = 0; q < 3; ++q) B[b][q] = kb[((t0 / 16 + b) * a.CK + ks) * 192 + 64 * q + lane];
    RowCubic rc;
    if constexpr (NT == 0) rc.start(r0, a.nxq);
    for (int r = r0; r < r1; r += 16) {
      const u32x4 *zr = za + ((int64_t)(r >> 4) * a.CK + ks) * 192 + lane;
      const u32x4 A[3] = {zr[0], zr[64], zr[128]};
      const f32x4 bv = bt[(r >> 4) * 64 + lane];
      // conj(k) z: Re = kr zr + ki zi, Im = kr zi - ki zr
      u32x4 Ai[3];
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) Ai[q][j] = __builtin_amdgcn_alignbit(A[q][j], A[q][j], 16) ^ 0x80000000u;
      f32x4 Mr[4], Mi[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        Mr[b] = mfma_3x3(A, B[b]);
        Mi[b] = mfma_3x3(Ai, B[b]);
      }
      // phases of this lane's sample at the 16 pixels, as turns reduced to
      // [-1/2, 1/2] before they are rounded to FP32
      float f[4][4];  // [pixel / 4][pixel % 4]
      if constexpr (NT == 0) {
        rc.expand(P, a.nx, a.ny, a.dx, a.dy, dx2, dx3);
        rc.next(a.nxq);
        rc.each([&](int i, double p) {
          const double ph = fma(P[10], uni[r + i], p);
          f[i >> 2][i & 3] = (float)(ph - __builtin_rint(ph));
        });
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const double *u = uni + (int64_t)(r + i) * NT;
          double ph = 0.0;
#pragma unroll
          for (int j = 0; j < NP; ++j) ph = fma(P[j], u[j], ph);
          f[i >> 2][i & 3] = (float)(ph - __builtin_rint(ph));
        }
      }
      float V[4][4];  // [sample block][register]
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        // (register: pixel quarter, lane quarter: sample block) transposed
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(f[0][v]), __float_as_uint(f[2][v]), false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(f[1][v]), __float_as_uint(f[3][v]), false, false);
        const auto p = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
        const auto q = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
        const float g[4] = {__uint_as_float(p[0]), __uint_as_float(p[1]), __uint_as_float(q[0]), __uint_as_float(q[1])};
        // Im(E M) = cos Mi + sin Mr
#pragma unroll
        for (int b = 0; b < 4; ++b)
          V[b][v] = fmaf(__builtin_amdgcn_cosf(g[b]), Mi[b][v], __builtin_amdgcn_sinf(g[b]) * Mr[b][v]);
      }
      if (a.gpart) {
        f32x4 S[2][4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int b = 0; b < 4; ++b)
            S[v >> 1][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                V[b][v], bv[v], v & 1 ? S[v >> 1][b] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int b = 0; b < 4; ++b) G[b] += S[0][b] + S[1][b];
      }
      if (a.dpart) {
        // over the 64 samples: blocks, then the 16 lanes of a row; a lane
        // keeps half of its four values at each of two stages and ends with
        // pixel 4 (lane / 16) + lane % 16 / 4
        float u[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
          u[v] = fmaf(V[0][v], tm[0], V[1][v] * tm[1]) + fmaf(V[2][v], tm[2], V[3][v] * tm[3]);
        const bool up8 = lane & 8, up4 = lane & 4;
        const float k0 = up8 ? u[2] : u[0], k1 = up8 ? u[3] : u[1];
        const float s0 = up8 ? u[0] : u[2], s1 = up8 ? u[1] : u[3];
        const float h0 = k0 + dpp<0x128>(s0), h1 = k1 + dpp<0x128>(s1);  // row_ror:8
        float h = (up4 ? h1 : h0) + dpp<0x141>(up4 ? h0 : h1);           // row_half_mirror
        h += dpp<0xb1>(h);                                               // quad_perm 1,0,3,2
        h += dpp<0x4e>(h);                                               // quad_perm 2,3,0,1
        if ((lane & 3) == 0) {
          float *o = &sdw[wave][r - r0 + 4 * (lane >> 4) + (l16 >> 2)];
          *o = ks ? *o + h : h;
        }
      }
    }
  }
  if (a.dpart) {
    __syncthreads();
    for (int i = threadIdx.x; i < r1 - r0; i += 256)
      a.dpart[(int64_t)rb * a.Rp + r0 + i] = (sdw[0][i] + sdw[1][i]) + (sdw[2][i] + sdw[3][i]);
  }
  if (a.gpart) {
    float *g = a.gpart + (int64_t)split * a.Tp * 16;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) g[(t0 + 16 * b + 4 * (lane >> 4) + v) * 16 + l16] = G[b][v];
  }
}

// grad_k[t][l] = -sum over pixel chunks, grad_dw[r] = -sum over 256-sample
// blocks, in FP64 and in order; the operand scales are divided out.
__global__ __launch_bounds__(256) void k_grad_reduce(const float *__restrict__ gpart, const float *__restrict__ dpart,
                                                     int64_t T, int64_t Tp, int L, int nsplit, int nx, int ny,
                                                     int nxq, int Rp, const float *__restrict__ amax,
                                                     double *__restrict__ gk, double *__restrict__ gd) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nk = gk ? T * L : 0, nd = gd ? (int64_t)nx * ny : 0;
  if (i >= nk + nd) return;
  const double inv =
      -1.0 / ((double)grad_scale(amax) * grad_scale(amax + kGradAmax) * grad_scale(amax + 2 * kGradAmax));
  const bool coef = i < nk;
  if (!coef) i -= nk;
  const float *p = coef ? gpart + (i / L) * 16 + i % L : dpart + (i / nx) * nxq + i % nx;
  const int64_t step = coef ? Tp * 16 : Rp;
  const int n = coef ? nsplit : (int)(Tp / 256);
  double s = 0.0;
  int k = 0;
  for (; k + 8 <= n; k += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(k + u) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; k < n; ++k) s += p[k * step];
  (coef ? gk : gd)[i] = inv * s;
}

struct GradLayout {
  EncPlan p;
  int chunk = 0, nsplit = 0, CK = 0;
  double *kap = nullptr, *bet = nullptr, *pmono = nullptr, *dwq = nullptr;
  u32x4 *za = nullptr, *kb = nullptr;
  float *tf = nullptr, *bt = nullptr, *amax = nullptr, *gpart = nullptr, *dpart = nullptr;
};

static int layout_grad(const expenc_op *op, int32_t precision, Arena &a, GradLayout *G) {
  // (the limit on ncoils * nbasis columns of the calls before is kept)
  const int L = op ? op->nbasis : 0;
  EX_TRY(make_plan(op, L > 0 ? L : 1, precision, &G->p));
  EX_TRY(make_plan(op, 1, precision, &G->p));
  const EncPlan &p = G->p;
  // chunks bound the length of an FP32 sum: kGradChunkMax products per
  // sample, fewer pixels where they hold several groups of 16 coils
  G->CK = (int)ceil_div(p.C, 16);
  const int cap = std::max(64, kGradChunkMax / G->CK / 16 * 16);
  G->chunk = default_chunk(p.Rp, p.Tp / 256, 1, 8, 2, 1.3, 1.5, 1.0, 16, cap, cap);
  G->nsplit = (int)ceil_div(p.Rp, G->chunk);
  if (p.sh) {
    G->pmono = a.take<double>(p.Tp * kPolyStride);
    G->dwq = a.take<double>(p.Rp);
  } else {
    G->kap = a.take<double>((size_t)p.Tp * p.NT);
    G->bet = a.take<double>((size_t)p.Rp * p.NT);
  }
  G->kb = a.take<u32x4>((size_t)p.Tp * G->CK * 12);
  G->za = a.take<u32x4>((size_t)p.Rp * G->CK * 12);
  G->tf = a.take<float>(p.Tp);
  G->bt = a.take<float>((size_t)p.Rp * 16);
  G->amax = a.take<float>(3 * kGradAmax);
  G->gpart = a.take<float>((size_t)G->nsplit * p.Tp * 16);
  G->dpart = a.take<float>((size_t)(p.Tp / 256) * p.Rp);
  return a.ok() ? EXPENC_OK : EXPENC_EWORKSPACE;
}

size_t grad_bytes(const expenc_op *op, int32_t precision) {
  Arena a;
  GradLayout G;
  if (layout_grad(op, precision, a, &G) != EXPENC_OK && !G.p.R) return 0;
  return a.used + 256;
}

}  // namespace expenc

using namespace expenc;

extern "C" int expenc_field_grad(const expenc_op *op, int32_t precision, const float *w, const float *kk,
                                 double *grad_coef, double *grad_dw0, void *ws, size_t ws_bytes, void *stream) {
  if (!w || !kk) return fail(EXPENC_EINVAL, "w or kk is NULL");
  if (precision != EXPENC_FP32) return fail(EXPENC_EUNSUPPORTED, "field gradients are computed in the FP32 form");
  GradLayout G;
  Arena a{static_cast<char *>(ws), ws_bytes, 0};
  const int st = layout_grad(op, precision, a, &G);
  if (st == EXPENC_EWORKSPACE || !ws)
    return fail(EXPENC_EWORKSPACE, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                grad_bytes(op, precision));
  EX_TRY(st);
  const EncPlan &p = G.p;
  if (op->nbasis < 1) grad_coef = nullptr;
  if (!grad_coef && !grad_dw0) return EXPENC_OK;
  hipStream_t s = (hipStream_t)stream;
  const float2 *w2 = reinterpret_cast<const float2 *>(w), *k2 = reinterpret_cast<const float2 *>(kk);
  EncBuffers eb;
  eb.kap = G.kap;
  eb.bet = G.bet;
  eb.pmono = G.pmono;
  eb.dwq = G.dwq;
  EX_TRY(enc_prepare(p, op, eb, s, kNeedForward));
  const float2 *s2 = reinterpret_cast<const float2 *>(op->smaps);
  k_grad_amax<<<dim3(kGradAmax, 3), 256, 0, s>>>(w2, p.R, k2, p.T, s2, p.C, G.amax);
  EX_LAUNCHED("gradient operand bounds");
  const GradPackArgs pa{k2, w2, s2, op->time, G.bet, G.amax, G.za, G.kb,
                        G.tf, G.bt, p.T, p.Tp, p.C, G.CK, p.NT, p.L, p.nx, p.ny, p.nxq, p.Rp, p.dx, p.dy, p.z0};
  k_grad_pack<<<(unsigned)ceil_div((p.Tp + p.Rp) * G.CK * 4 + p.Tp + p.Rp, 256), 256, 0, s>>>(pa);
  EX_LAUNCHED("gradient operands");
  const GradArgs ga{grad_coef ? G.gpart : nullptr, grad_dw0 ? G.dpart : nullptr, p.Tp, p.Rp, G.CK, p.ny, p.nx,
                    p.nxq, G.chunk, G.nsplit, p.dx, p.dy};
  const f32x4 *bt = reinterpret_cast<const f32x4 *>(G.bt);
  const unsigned grid = split_grid(p.Tp / 256 * G.nsplit);
  if (p.sh) k_field_grad<0><<<grid, 256, 0, s>>>(G.pmono, G.dwq, G.za, G.kb, G.tf, bt, ga);
  else if (p.NT == 4) k_field_grad<4><<<grid, 256, 0, s>>>(G.kap, G.bet, G.za, G.kb, G.tf, bt, ga);
  else if (p.NT == 10) k_field_grad<10><<<grid, 256, 0, s>>>(G.kap, G.bet, G.za, G.kb, G.tf, bt, ga);
  else k_field_grad<17><<<grid, 256, 0, s>>>(G.kap, G.bet, G.za, G.kb, G.tf, bt, ga);
  EX_LAUNCHED("field gradient");
  const int64_t n = (grad_coef ? p.T * p.L : 0) + (grad_dw0 ? (int64_t)p.R : 0);
  k_grad_reduce<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(G.gpart, G.dpart, p.T, p.Tp, p.L, G.nsplit, p.nx, p.ny,
                                                           p.nxq, p.Rp, G.amax, grad_coef, grad_dw0);
  EX_LAUNCHED("gradient sums");
  return EXPENC_OK;
}
