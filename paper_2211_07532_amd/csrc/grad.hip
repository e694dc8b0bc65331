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

namespace expenc {

constexpr int kGradTerms = 32;      // columns of the basis table (L <= 16 used)
constexpr int kGradChunkMax = 1024; // pixels one workgroup accumulates in FP32
constexpr int kGradAmax = 64;       // workgroups of the magnitude pre-pass per array

// Per-workgroup max component magnitude of w [R] (blockIdx.y 0) and kk [n]
// (blockIdx.y 1) into amax[2][kGradAmax].
__global__ __launch_bounds__(256) void k_grad_amax(const float2 *__restrict__ w, int64_t R,
                                                   const float2 *__restrict__ kk, int64_t n,
                                                   float *__restrict__ amax) {
  __shared__ float wm[4];
  const float2 *v = blockIdx.y ? kk : w;
  const int64_t m = blockIdx.y ? n : R;
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
// for an all-zero or non-finite array): M is a product of kk and w in FP32,
// and with both scaled it neither overflows nor underflows for any inputs.
// The reductions divide the scales out in FP64.
__device__ inline float grad_scale(const float *__restrict__ amax) {
  float m = 0.f;
  for (int i = 0; i < kGradAmax; ++i) m = fmaxf(m, amax[i]);
  if (!(m > 0.f) || !(m <= 3.0e38f)) return 1.f;
  int e;
  (void)frexpf(m, &e);
  return ldexpf(1.f, min(126, max(-126, -e)));
}

// Operands of the gradient contraction: kkt[c][re | im][Tp] = scaled kk
// (transposed, so the lanes of a wave read consecutive samples), tf[Tp] the
// sample times, bt[Rp][kGradTerms] = b_l at the padded pixels (from the
// table bet [Rp][NT], or the solid harmonics at the pixel centre), ws[Rp] the
// scaled w; zero on padding.  One element per thread, array by array.
__global__ __launch_bounds__(256) void k_grad_pack(const float2 *__restrict__ kk, const double *__restrict__ time,
                                                   int64_t T, int64_t Tp, int C, const double *__restrict__ bet,
                                                   int NT, int L, const float2 *__restrict__ w, int nx, int ny,
                                                   int nxq, int Rp, double dx, double dy, double z0,
                                                   const float *__restrict__ amax, float *__restrict__ kkt,
                                                   float *__restrict__ tf, float *__restrict__ bt,
                                                   float2 *__restrict__ wsc) {
  int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < Tp * C) {
    const int64_t t = i % Tp, c = i / Tp;
    float2 v = make_float2(0.f, 0.f);
    if (t < T) {
      const float s = grad_scale(amax + kGradAmax);
      v = kk[t * C + c];
      v.x *= s;
      v.y *= s;
    }
    kkt[2 * c * Tp + t] = v.x;
    kkt[(2 * c + 1) * Tp + t] = v.y;
    return;
  }
  i -= Tp * C;
  if (i < Tp) {
    tf[i] = i < T ? (float)time[i] : 0.f;
    return;
  }
  i -= Tp;
  if (i >= Rp) return;
  const int r = (int)i, yy = r / nxq, xx = r % nxq;
  const bool in = xx < nx && yy < ny;
  float2 u = make_float2(0.f, 0.f);
  if (in) {
    const float s = grad_scale(amax);
    u = w[(int64_t)yy * nx + xx];
    u.x *= s;
    u.y *= s;
  }
  wsc[r] = u;
  double v[16];
  if (!bet) sh_eval((xx - 0.5 * nx) * dx, (yy - 0.5 * ny) * dy, z0, v);
#pragma unroll
  for (int l = 0; l < kGradTerms; ++l) {
    float b = 0.f;
    if (in && l < L) b = (float)(bet ? bet[(int64_t)r * NT + min(l, NT - 1)] : v[l & 15]);
    bt[(int64_t)r * kGradTerms + l] = b;
  }
}

// Arguments of the gradient contraction.
struct GradArgs {
  const double *kap, *bet;      // maps kind: [Tp][NT], [Rp][NT]
  const double *pmono, *dwq;    // solid-harmonic kind: [Tp][kPolyStride], [Rp]
  const float *kkt, *tf, *bt;
  const float2 *ws, *smaps;
  float *gpart, *dpart;         // [nsplit][Tp][16], [Tp/256][Rp]; NULL: that gradient is not wanted
  int64_t Tp;
  int Rp, C, R, nx, ny, nxq, chunk, nsplit;
  double dx, dy;
};

// One workgroup: 256 samples (64 per wave) x a chunk of pixels, in blocks of
// 32 pixels.  Per block a wave forms M^T (rows: pixels, columns: samples) on
// v_mfma_f32_32x32x2_f32 over coils, its two K indices being the real and the
// imaginary part of a coil; evaluates the phases as the FP32 forward does
// (its own sample, two wave-uniform pixels at a time, FP64, exchanged by
// v_permlane32_swap); and multiplies.  V then sits with its sample in the
// lane and its pixel in the register, which is the A-operand layout of the
// product with the basis table, so grad_k is accumulated on the matrix cores
// without moving V.  grad_dw sums over lanes by recursive halving.
// Bound: the FP32 matrix cores (4 C + 32 products per entry) plus the FP64
// phase, which does not co-issue with them.  At 128 x 128, 16 coils, T = 12000
// and 16 terms 0.68 ms, where the basis-weighted forward and the adjoint took
// 3.78 + 0.34 ms.
// NT 0: solid-harmonic kind (polynomial phase); else the general basis.
template <int NT>
__global__ __launch_bounds__(256, 2) void k_field_grad(GradArgs a) {
  __shared__ float sdw[2][4][32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  int split, rb;
  if (!split_tile(blockIdx.x, (int)(a.Tp / 256), a.nsplit, &split, &rb)) return;
  const int64_t t0 = (int64_t)rb * 256 + wave * 64;
  constexpr int NP = NT ? NT : 11;
  double P[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) P[j] = NT ? a.kap[(t0 + lane) * NT + j] : a.pmono[(t0 + lane) * kPolyStride + j];
  const float tm0 = a.tf[t0 + l32], tm1 = a.tf[t0 + 32 + l32];
  const double dx2 = a.dx * a.dx, dx3 = dx2 * a.dx;
  const float *kb = a.kkt + half * a.Tp + t0 + l32;  // this lane's K row (re or im) at its samples
  f32x16 G[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) G[b][v] = 0.f;
  const int r0 = split * a.chunk, r1 = min(a.Rp, r0 + a.chunk);
  int par = 0;
  for (int r = r0; r < r1; r += 32, par ^= 1) {
    // this lane's pixel as a row of M^T (padding: w is zero there)
    const int rq = r + l32, py = rq / a.nxq, px = rq - py * a.nxq;
    const int pix = min(py, a.ny - 1) * a.nx + min(px, a.nx - 1);
    const float2 w = a.ws[rq];
    const float2 *sp = a.smaps + pix;
    f32x16 Mr[2], Mi[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) Mr[b][v] = Mi[b][v] = 0.f;
#pragma unroll 4
    for (int c = 0; c < a.C; ++c) {
      const float2 s = sp[(int64_t)c * a.R];
      const float zr = s.x * w.x - s.y * w.y, zi = s.x * w.y + s.y * w.x;
      const float k0 = kb[2 * c * a.Tp], k1 = kb[2 * c * a.Tp + 32];
      // conj(k) z: Re = kr zr + ki zi, Im = kr zi - ki zr
      const float ar = half ? zi : zr, ai = half ? -zr : zi;
      Mr[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, k0, Mr[0], 0, 0, 0);
      Mi[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, k0, Mi[0], 0, 0, 0);
      Mr[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, k1, Mr[1], 0, 0, 0);
      Mi[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, k1, Mi[1], 0, 0, 0);
    }
    const float *bp = a.bt + (int64_t)(r + 4 * half) * kGradTerms + l32;
    float u[16];
    double c0 = 0, d1 = 0, d2 = 0, d3 = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int pa_ = 8 * (v >> 2) + (v & 3), pb_ = pa_ + 4;  // pixels of the two half-waves' rows
      double pa, pb;
      if constexpr (NT == 0) {
        if ((v & 7) == 0) {
          // row polynomial of this 16-pixel tile around its centre
          const int rt = r + 2 * v, yi = rt / a.nxq, xi = rt - yi * a.nxq + 8;
          const double ym = (yi - 0.5 * a.ny) * a.dy, xc = (xi - 0.5 * a.nx) * a.dx;
          const double a0 = P[0] + ym * (P[2] + ym * (P[5] + ym * P[9]));
          const double a1 = P[1] + ym * (P[4] + ym * P[8]);
          const double a2 = P[3] + ym * P[7], a3 = P[6];
          c0 = a0 + xc * (a1 + xc * (a2 + xc * a3));
          d1 = (a1 + xc * (2.0 * a2 + 3.0 * a3 * xc)) * a.dx;
          d2 = (a2 + 3.0 * a3 * xc) * dx2;
          d3 = a3 * dx3;
        }
        const double ka = (pa_ & 15) - 8, kb_ = (pb_ & 15) - 8;
        pa = fma(P[10], a.dwq[r + pa_], fma(fma(fma(d3, ka, d2), ka, d1), ka, c0));
        pb = fma(P[10], a.dwq[r + pb_], fma(fma(fma(d3, kb_, d2), kb_, d1), kb_, c0));
      } else {
        const double *ba = a.bet + (int64_t)(r + pa_) * NT;
        pa = pb = 0.0;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
          pa = fma(P[j], ba[j], pa);
          pb = fma(P[j], ba[4 * NT + j], pb);
        }
      }
      // centred reduction to [-1/2, 1/2] turns before rounding to FP32
      const float fa = (float)(pa - __builtin_rint(pa)), fb = (float)(pb - __builtin_rint(pb));
      const float ca = __builtin_amdgcn_cosf(fa), sa = __builtin_amdgcn_sinf(fa);
      const float cb = __builtin_amdgcn_cosf(fb), sb = __builtin_amdgcn_sinf(fb);
      const auto cc = __builtin_amdgcn_permlane32_swap(__float_as_uint(ca), __float_as_uint(cb), false, false);
      const auto ss = __builtin_amdgcn_permlane32_swap(__float_as_uint(sa), __float_as_uint(sb), false, false);
      // Im(E M) = cos Mi + sin Mr
      const float v0 = fmaf(__uint_as_float(cc[0]), Mi[0][v], __uint_as_float(ss[0]) * Mr[0][v]);
      const float v1 = fmaf(__uint_as_float(cc[1]), Mi[1][v], __uint_as_float(ss[1]) * Mr[1][v]);
      if (a.gpart) {
        const float b = bp[pa_ * kGradTerms];
        G[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v0, b, G[0], 0, 0, 0);
        G[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(v1, b, G[1], 0, 0, 0);
      }
      u[v] = fmaf(v0, tm0, v1 * tm1);
    }
    if (a.dpart) {
      // sum over the 32 samples (lanes) of each half: at each stage a lane
      // keeps one half of its values; lane l ends with element v = (l%32)/2
#pragma unroll
      for (int o = 16, n = 16; o > 1; o >>= 1, n >>= 1) {
        const bool up = (lane & o) != 0;
#pragma unroll
        for (int i = 0; i < n / 2; ++i) {
          const float keep = up ? u[i + n / 2] : u[i], send = up ? u[i] : u[i + n / 2];
          u[i] = keep + __shfl_xor(send, o);
        }
      }
      u[0] += __shfl_xor(u[0], 1);
      if ((lane & 1) == 0) {
        const int v = l32 >> 1;
        sdw[par][wave][8 * (v >> 2) + 4 * half + (v & 3)] = u[0];
      }
      __syncthreads();
      // (the other buffer is written next; its readers passed this barrier)
      if (threadIdx.x < 32)
        a.dpart[(int64_t)rb * a.Rp + r + threadIdx.x] = (sdw[par][0][threadIdx.x] + sdw[par][1][threadIdx.x]) +
                                                        (sdw[par][2][threadIdx.x] + sdw[par][3][threadIdx.x]);
    }
  }
  if (a.gpart && l32 < 16) {
    float *g = a.gpart + (int64_t)split * a.Tp * 16;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        g[(t0 + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3)) * 16 + l32] = G[b][v];
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
  const double inv = -1.0 / ((double)grad_scale(amax) * grad_scale(amax + kGradAmax));
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
  int chunk = 0, nsplit = 0;
  double *kap = nullptr, *bet = nullptr, *pmono = nullptr, *dwq = nullptr;
  float *kkt = nullptr, *tf = nullptr, *bt = nullptr, *amax = nullptr, *gpart = nullptr,
        *dpart = nullptr;
  float2 *wsc = nullptr;
};

static int layout_grad(const expenc_op *op, int32_t precision, Arena &a, GradLayout *G) {
  // (the limit on ncoils * nbasis columns of the calls before is kept)
  const int L = op ? op->nbasis : 0;
  EX_TRY(make_plan(op, L > 0 ? L : 1, precision, &G->p));
  EX_TRY(make_plan(op, 1, precision, &G->p));
  const EncPlan &p = G->p;
  // about 1024 workgroups: two rounds of the two a CU holds; chunks of at
  // most kGradChunkMax pixels bound the length of an FP32 sum
  const int64_t nrb = p.Tp / 256;
  const int64_t want = std::max<int64_t>(ceil_div(1024, nrb), ceil_div(p.Rp, kGradChunkMax));
  G->chunk = (int)round_up(ceil_div(p.Rp, std::min<int64_t>(want, p.Rp / 32)), 32);
  G->nsplit = (int)ceil_div(p.Rp, G->chunk);
  if (p.sh) {
    G->pmono = a.take<double>(p.Tp * kPolyStride);
    G->dwq = a.take<double>(p.Rp);
  } else {
    G->bet = a.take<double>((size_t)p.Rp * p.NT);
  }
  G->kap = a.take<double>(p.Tp * p.NT);
  G->kkt = a.take<float>(2 * p.Tp * p.C);
  G->tf = a.take<float>(p.Tp);
  G->bt = a.take<float>((size_t)p.Rp * kGradTerms);
  G->wsc = a.take<float2>(p.Rp);
  G->amax = a.take<float>(2 * kGradAmax);
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
  k_grad_amax<<<dim3(kGradAmax, 2), 256, 0, s>>>(w2, p.R, k2, p.T * p.C, G.amax);
  EX_LAUNCHED("gradient operand bounds");
  k_grad_pack<<<(unsigned)ceil_div(p.Tp * p.C + p.Tp + p.Rp, 256), 256, 0, s>>>(
      k2, op->time, p.T, p.Tp, p.C, G.bet, p.NT, p.L, w2, p.nx, p.ny, p.nxq, p.Rp, p.dx, p.dy, p.z0, G.amax, G.kkt,
      G.tf, G.bt, G.wsc);
  EX_LAUNCHED("gradient operands");
  const GradArgs ga{G.kap, G.bet, G.pmono, G.dwq, G.kkt, G.tf, G.bt, G.wsc,
                    reinterpret_cast<const float2 *>(op->smaps), grad_coef ? G.gpart : nullptr,
                    grad_dw0 ? G.dpart : nullptr, p.Tp, p.Rp, p.C, p.R, p.nx, p.ny, p.nxq, G.chunk, G.nsplit,
                    p.dx, p.dy};
  const unsigned grid = split_grid(p.Tp / 256 * G.nsplit);
  if (p.sh) k_field_grad<0><<<grid, 256, 0, s>>>(ga);
  else if (p.NT == 4) k_field_grad<4><<<grid, 256, 0, s>>>(ga);
  else if (p.NT == 10) k_field_grad<10><<<grid, 256, 0, s>>>(ga);
  else k_field_grad<17><<<grid, 256, 0, s>>>(ga);
  EX_LAUNCHED("field gradient");
  const int64_t n = (grad_coef ? p.T * p.L : 0) + (grad_dw0 ? (int64_t)p.R : 0);
  k_grad_reduce<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(G.gpart, G.dpart, p.T, p.Tp, p.L, G.nsplit, p.nx, p.ny,
                                                           p.nxq, p.Rp, G.amax, grad_coef, grad_dw0);
  EX_LAUNCHED("gradient sums");
  return EXPENC_OK;
}
