// Coil pre-whitening and coil compression (Methods 2.2.1: k-space data
// compressed to virtual coils for speed, receiver noise correlation removed
// by pre-whitening).
//
// Pre-whitening: Psi = L L^H (Cholesky, FP64, one workgroup), then every coil
// vector (one per sample of y, one per pixel of the maps) is replaced by
// L^{-1} v by forward substitution.
//
// Compression: the coil Gram matrix G = Y^H Y over all samples (FP64 partial
// sums per block of samples, summed in a fixed order), its eigenvectors by a
// cyclic Jacobi method in one workgroup (complex Hermitian rotations, the
// pairs of a sweep scheduled round-robin so that C/2 disjoint rotations run
// at once, everything in LDS), sorted by eigenvalue descending; then
// y_v = Y V_k and the virtual maps S_v[j] = sum_c V[c][j] S_c.
//
// The factorisations are serial chains in one workgroup, bound by the latency
// of FP64 roots and divisions, LDS and barriers.  Rotation phases of
// converged pairs follow the last bits of G, so the arithmetic of every step
// is kept as it is to the bit.  32 coils, 16384 samples, 148 x 148 maps, 20
// virtual coils: Jacobi 900 -> 348 us, Cholesky 85 -> 25, whitening 163 -> 76,
// Gram matrix 68 -> 24, compression 31 -> 24.
#include <cmath>

#include "internal.h"

namespace expenc {

namespace {

constexpr int kMaxCoils = 64;
constexpr int kGramChunk = 128;  // samples per Gram partial

constexpr int kWhitenRows = 8;   // components solved together
__host__ __device__ inline int padded_rows(int C) { return (C + kWhitenRows - 1) / kWhitenRows * kWhitenRows; }

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// part[blk][o] = sum over the block's samples of conj(y[t][a]) y[t][b], o the
// place of (a, b), a <= b, in the rows of the upper triangle (G is
// Hermitian); one product per thread, blockIdx.y a range of 256 of them.
__global__ __launch_bounds__(256) void k_gram_part(const float2 *__restrict__ y, int64_t T, int C,
                                                   double2 *__restrict__ part) {
  extern __shared__ float2 ys[];  // [kGramChunk][C]
  const int64_t t0 = (int64_t)blockIdx.x * kGramChunk;
  const int nt = (int)min<int64_t>(kGramChunk, T - t0);
  for (int i = threadIdx.x; i < nt * C; i += 256) ys[i] = y[t0 * C + i];
  __syncthreads();
  const int o = blockIdx.y * 256 + threadIdx.x, no = C * (C + 1) / 2;
  if (o >= no) return;
  int a = 0, left = o;
  while (left >= C - a) left -= C - a++;
  const float2 *pa = ys + a, *pb = ys + a + left;
  double sr = 0.0, si = 0.0;
#pragma unroll 8
  for (int t = 0; t < nt; ++t) {
    const float2 u = pa[t * C], v = pb[t * C];
    sr += (double)u.x * v.x + (double)u.y * v.y;
    si += (double)u.x * v.y - (double)u.y * v.x;
  }
  part[(int64_t)blockIdx.x * no + o] = make_double2(sr, si);
}

// Sums of the partials in block order, eight loads in flight; fills both
// triangles.
__global__ __launch_bounds__(64) void k_gram_sum(const double2 *__restrict__ part, int nblk, int C,
                                                 double2 *__restrict__ g) {
  const int no = C * (C + 1) / 2, o = blockIdx.x * 64 + threadIdx.x;
  if (o >= no) return;
  double sr = 0.0, si = 0.0;
  int b = 0;
  for (; b + 8 <= nblk; b += 8) {
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(b + u) * no + o];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      sr += v[u].x;
      si += v[u].y;
    }
  }
  for (; b < nblk; ++b) {
    const double2 v = part[(int64_t)b * no + o];
    sr += v.x;
    si += v.y;
  }
  int a = 0, left = o;
  while (left >= C - a) left -= C - a++;
  const int c = a + left;
  g[a * C + c] = make_double2(sr, si);
  g[c * C + a] = make_double2(sr, -si);
}

// Eigen-decomposition of the Hermitian C x C matrix g: eigenvalues
// descending to w, eigenvectors as the columns of v ([C][C] row-major).
//
// A round rotates the C/2 disjoint pairs at once, A <- U^H A U and V <- V U:
// the 2 x 2 block of rows (p, q) of one pair and columns (p', q') of another
// depends on those four values alone, so a thread takes whole blocks, rows
// first, then columns, in registers.  V is not needed for the next round's
// angles, so the first wave evaluates those (a chain of FP64 roots and
// divisions) while the others apply the last round to V; a round has two
// barriers.  Rows are padded by one value: the threads of V's update walk
// down a column, which at a row stride of 512 bytes put them all on one LDS
// bank.
constexpr int kJacobiThreads = 576;  // one wave of angles and 512 threads of V's update
struct JacobiRound {
  double2 cs[kMaxCoils / 2], ph[kMaxCoils / 2];  // (c, s) and e of each pair
};

// Pair j of round r of n players (round robin): p < q.
__device__ inline void jacobi_pair(int r, int j, int n, int &p, int &q) {
  if (j == 0) {
    p = r;
    q = n - 1;
    return;
  }
  p = r + j;
  if (p >= n - 1) p -= n - 1;
  q = r - j;
  if (q < 0) q += n - 1;
  if (p > q) {
    const int t = p;
    p = q;
    q = t;
  }
}

// (xp, xq) <- (c xp - s t, s xp + c t) with t = e xq (rows p, q of U^H A) or
// conj(e) xq (columns p, q of A U and V U).  The fused operations are written
// out: their choice decides the last bits.
template <bool ROWS>
__device__ inline void rotate(double c, double s, double2 e, double2 &xp, double2 &xq) {
  const double tx = ROWS ? fma(e.x, xq.x, -(e.y * xq.y)) : fma(e.x, xq.x, e.y * xq.y);
  const double ty = ROWS ? fma(e.y, xq.x, e.x * xq.y) : fma(e.x, xq.y, -(e.y * xq.x));
  const double2 np = make_double2(fma(c, xp.x, -(s * tx)), fma(c, xp.y, -(s * ty)));
  xq = make_double2(fma(s, xp.x, c * tx), fma(s, xp.y, c * ty));
  xp = np;
}

__global__ __launch_bounds__(kJacobiThreads) void k_jacobi(const double2 *__restrict__ g, int C, int max_sweeps,
                                                           double2 *__restrict__ v_out, double *__restrict__ w_out,
                                                           unsigned *status) {
  extern __shared__ double2 sh[];
  const int S = C + 1;      // row stride
  double2 *A = sh;          // [C][S]
  double2 *V = sh + C * S;  // [C][S]
  __shared__ JacobiRound rot[2];
  __shared__ double red[2][256];
  __shared__ int perm[kMaxCoils];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int i = tid; i < C * C; i += kJacobiThreads) {
    A[i / C * S + i % C] = g[i];
    V[i / C * S + i % C] = make_double2((i / C) == (i % C) ? 1.0 : 0.0, 0.0);
  }
  const int n = C + (C & 1);  // players of the round-robin schedule (one dummy when C is odd)
  const int np = n / 2;
  auto angles = [&](int r, JacobiRound &R) {
    if (tid >= np) return;
    int p, q;
    jacobi_pair(r, tid, n, p, q);
    double c = 1.0, s = 0.0;
    double2 ph = make_double2(1.0, 0.0);
    if (q < C) {
      const double2 gpq = A[p * S + q];
      const double m = sqrt(fma(gpq.x, gpq.x, gpq.y * gpq.y));
      const double a = A[p * S + p].x, b = A[q * S + q].x;
      if (m > 1e-300 && m > 1e-18 * (fabs(a) + fabs(b))) {
        // real Jacobi rotation of [[a, m], [m, b]]; the phase of g_pq is
        // removed by diag(1, e^{-i phi}) on index q
        const double th = (b - a) / (2.0 * m);
        const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(fma(th, th, 1.0)));
        c = 1.0 / sqrt(fma(t, t, 1.0));
        s = t * c;
        ph = make_double2(gpq.x / m, gpq.y / m);
      }
    }
    R.cs[tid] = make_double2(c, s);
    R.ph[tid] = ph;
  };
  // V <- V U of round r: a column of threads per pair (all but the first wave)
  const int vt = tid - 64, vrow = vt % C, vpair = vt / C, vstep = (kJacobiThreads - 64) / C;
  auto update_v = [&](int r, const JacobiRound &R) {
    if (vt < 0 || vpair >= vstep) return;
    for (int l = vpair; l < np; l += vstep) {
      int p, q;
      jacobi_pair(r, l, n, p, q);
      const double2 cs = R.cs[l];
      if (q >= C || cs.y == 0.0) continue;
      double2 vp = V[vrow * S + p], vq = V[vrow * S + q];
      rotate<false>(cs.x, cs.y, R.ph[l], vp, vq);
      V[vrow * S + p] = vp;
      V[vrow * S + q] = vq;
    }
  };
  // A <- U^H A U of round r: block (rows of pair k, columns of pair l) per item
  const int ak = tid / np, al = tid % np, astep = kJacobiThreads / np;
  auto update_a = [&](int r, const JacobiRound &R) {
    if (ak >= astep) return;
    int pl, ql;
    jacobi_pair(r, al, n, pl, ql);
    const double2 csl = R.cs[al], el = R.ph[al];
    const bool cl = ql < C;
    for (int k = ak; k < np; k += astep) {
      int pk, qk;
      jacobi_pair(r, k, n, pk, qk);
      const bool rk = qk < C;
      const double2 zero = make_double2(0.0, 0.0);
      const double2 csk = R.cs[k], ek = R.ph[k];
      double2 x00 = A[pk * S + pl], x01 = cl ? A[pk * S + ql] : zero;
      double2 x10 = rk ? A[qk * S + pl] : zero, x11 = rk && cl ? A[qk * S + ql] : zero;
      if (rk && csk.y != 0.0) {
        rotate<true>(csk.x, csk.y, ek, x00, x10);
        rotate<true>(csk.x, csk.y, ek, x01, x11);
      }
      if (cl && csl.y != 0.0) {
        rotate<false>(csl.x, csl.y, el, x00, x01);
        rotate<false>(csl.x, csl.y, el, x10, x11);
      }
      A[pk * S + pl] = x00;
      if (cl) A[pk * S + ql] = x01;
      if (rk) A[qk * S + pl] = x10;
      if (rk && cl) A[qk * S + ql] = x11;
    }
  };
  __syncthreads();
  int par = 0, last = -1;  // last: the round (in rot[par ^ 1]) that V has not had yet
  for (int sweep = 0; sweep < max_sweeps; ++sweep) {
    // convergence test on the off-diagonal mass: 256 strided sums, added as a
    // binary tree (lane i and i + 128, + 64, ...)
    double off = 0.0, tot = 0.0;
    if (tid < 256) {
      for (int i = tid; i < C * C; i += 256) {
        const double2 a = A[i / C * S + i % C];
        const double m = fma(a.x, a.x, a.y * a.y);
        tot += m;
        if (i / C != i % C) off += m;
      }
      red[0][tid] = off;
      red[1][tid] = tot;
    }
    __syncthreads();
    off = (red[0][lane] + red[0][lane + 128]) + (red[0][lane + 64] + red[0][lane + 192]);
    tot = (red[1][lane] + red[1][lane + 128]) + (red[1][lane + 64] + red[1][lane + 192]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      off += __shfl_down(off, o);
      tot += __shfl_down(tot, o);
    }
    off = __shfl(off, 0);
    tot = __shfl(tot, 0);
    if (!(off > 1e-30 * tot)) break;  // (uniform: every wave adds the same values)
    for (int r = 0; r < n - 1; ++r, par ^= 1) {
      if (tid < 64) angles(r, rot[par]);
      else if (last >= 0) update_v(last, rot[par ^ 1]);
      __syncthreads();
      update_a(r, rot[par]);
      last = r;
      __syncthreads();
    }
  }
  if (last >= 0) update_v(last, rot[par ^ 1]);
  __syncthreads();
  // eigenvalues descending (ties keep index order): the place of i is the
  // number of eigenvalues before it; status: any non-finite
  if (tid == 0) status[0] = 0u;
  if (tid < C) perm[tid] = tid;
  __syncthreads();
  if (tid < C) {
    const double d = A[tid * S + tid].x;
    if (!isfinite(d)) atomicOr(status, kStatusNonFinite);
    int place = 0;
    for (int j = 0; j < C; ++j) {
      const double e = A[j * S + j].x;
      place += e > d || (e == d && j < tid);
    }
    perm[place] = tid;
  }
  __syncthreads();
  for (int i = tid; i < C; i += kJacobiThreads)
    if (w_out) w_out[i] = A[perm[i] * S + perm[i]].x;
  for (int i = tid; i < C * C; i += kJacobiThreads) v_out[i] = V[i / C * S + perm[i % C]];
}

// Reads the coil vectors k0 .. k0 + 63 (component c of vector k at
// in[k * vs + c * cs]; zero from vector n on) and hands each value to
// put(c, vector, value): NT threads along the array's contiguous axis, eight
// loads in flight per thread.
template <int NT, class Put>
__device__ inline void stage_vectors(const float2 *in, int64_t vs, int64_t cs, int C, int64_t k0, int64_t n, Put put) {
  const int nv = (int)min<int64_t>(64, n - k0);
  for (int base = threadIdx.x; base < 64 * C; base += 8 * NT) {
    float2 u[8];
    int v[8], c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int i = base + j * NT;
      v[j] = cs == 1 ? i / C : i & 63;
      c[j] = cs == 1 ? i - v[j] * C : i >> 6;
      u[j] = i < 64 * C && v[j] < nv ? in[(k0 + v[j]) * vs + c[j] * cs] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (base + j * NT < 64 * C) put(c[j], v[j], u[j]);
  }
}

// out[j] = sum_c V[c][j] in[c] for n coil vectors, j < nout: component c of
// vector k at in[k * ivs + c * ics], result j at out[k * ovs + j * ocs].  64
// vectors (one per lane) per workgroup, staged in LDS as [c][vector], V beside
// them as [j][c]; the four waves take the result components in turn.
__global__ __launch_bounds__(256) void k_compress(const double2 *__restrict__ V, int C, int nout,
                                                  const float2 *__restrict__ in, int64_t ivs, int64_t ics,
                                                  float2 *__restrict__ out, int64_t ovs, int64_t ocs, int64_t n) {
  extern __shared__ double2 vt[];                          // [nout][C]
  float2 *const xs = reinterpret_cast<float2 *>(vt + nout * C);  // [C][65]
  const int64_t k0 = (int64_t)blockIdx.x * 64;
  for (int i = threadIdx.x; i < nout * C; i += 256) vt[i] = V[i % C * C + i / C];
  stage_vectors<256>(in, ivs, ics, C, k0, n, [&](int c, int v, float2 u) { xs[c * 65 + v] = u; });
  __syncthreads();
  const int lane = threadIdx.x & 63;
  for (int j = threadIdx.x >> 6; j < nout; j += 4) {
    const double2 *row = vt + j * C;
    double sr = 0.0, si = 0.0;
#pragma unroll 4
    for (int c = 0; c < C; ++c) {
      const float2 a = xs[c * 65 + lane];
      const double2 b = row[c];
      sr += a.x * b.x - a.y * b.y;
      si += a.x * b.y + a.y * b.x;
    }
    if (k0 + lane < n) out[(k0 + lane) * ovs + j * ocs] = make_float2((float)sr, (float)si);
  }
}

// Lt = L^T ([C][round_up(C, kWhitenRows)], zero above the diagonal of L and
// on the padding) with L L^H = psi; NaN when psi is not positive definite.
// Right-looking: step k divides column k by the pivot and subtracts its outer
// product from the trailing block (the subtractions of an entry in the order
// of k).  status[0] = kStatusNonFinite when a pivot is not positive or not
// finite, else 0.
__global__ __launch_bounds__(512) void k_cholesky(const double2 *__restrict__ psi, int C, double2 *__restrict__ Lt,
                                                  unsigned *status) {
  extern __shared__ double2 a[];  // [C][C + 1]
  const int S = C + 1;
  __shared__ int bad;
  const int tid = threadIdx.x;
  if (tid == 0) bad = 0;
  for (int i = tid; i < C * C; i += 512) a[i / C * S + i % C] = psi[i];
  __syncthreads();
  for (int k = 0; k < C; ++k) {
    const double d = a[k * S + k].x;
    const double diag = sqrt(d);  // NaN for a non-positive pivot
    if (tid == 0 && (!(d > 0.0) || !isfinite(d))) bad = 1;
    if (tid > k && tid < C) {
      const double2 v = a[tid * S + k];
      a[tid * S + k] = make_double2(v.x / diag, v.y / diag);
    }
    __syncthreads();
    if (tid == 0) a[k * S + k] = make_double2(diag, 0.0);
    for (int i = tid; i < (C - 1 - k) * C; i += 512) {
      const int r = k + 1 + i / C, c = i % C;
      if (c <= k || c > r) continue;
      const double2 lr = a[r * S + k];
      if (c == r) {
        a[r * S + r].x -= lr.x * lr.x + lr.y * lr.y;
      } else {
        const double2 t = cmul(lr, cconj(a[c * S + k]));
        a[r * S + c].x -= t.x;
        a[r * S + c].y -= t.y;
      }
    }
    __syncthreads();
  }
  const int Cp = padded_rows(C);
  for (int i = tid; i < C * Cp; i += 512) {
    const int m = i / Cp, r = i - m * Cp;
    Lt[i] = r >= m && r < C ? a[r * S + m] : make_double2(0.0, 0.0);
  }
  if (tid == 0) status[0] = bad ? kStatusNonFinite : 0u;
}

// v <- L^{-1} v for n coil vectors v_k[c] = x[k * vs + c * cs], by forward
// substitution.  One wave per workgroup, one vector per lane; solved
// components are kept in LDS as [c][lane], padded (a per-lane array indexed at run
// time would live in scratch memory).  kWhitenRows components are solved at a
// time, so each earlier one is read once for all of them and their sums are
// independent chains; L is staged too (read from memory, its entries cost the
// lone wave a latency each).
__global__ __launch_bounds__(64) void k_whiten(const double2 *__restrict__ Lt, int C, float2 *x, int64_t n, int64_t vs,
                                               int64_t cs) {
  extern __shared__ double2 w[];  // [C][65], then L^T
  const int lane = threadIdx.x, Cp = padded_rows(C);
  const int64_t k0 = (int64_t)blockIdx.x * 64;
  double2 *const lt = w + C * 65;
#pragma unroll 8
  for (int i = lane; i < C * Cp; i += 64) lt[i] = Lt[i];
  stage_vectors<64>(x, vs, cs, C, k0, n, [&](int c, int v, float2 u) { w[c * 65 + v] = make_double2(u.x, u.y); });
  __syncthreads();
  for (int i0 = 0; i0 < C; i0 += kWhitenRows) {
    double2 s[kWhitenRows];
#pragma unroll
    for (int j = 0; j < kWhitenRows; ++j) s[j] = i0 + j < C ? w[(i0 + j) * 65 + lane] : make_double2(0.0, 0.0);
    for (int m = 0; m < i0; ++m) {
      const double2 u = w[m * 65 + lane];
#pragma unroll
      for (int j = 0; j < kWhitenRows; ++j) {
        const double2 t = cmul(lt[m * Cp + i0 + j], u);
        s[j].x -= t.x;
        s[j].y -= t.y;
      }
    }
#pragma unroll
    for (int j = 0; j < kWhitenRows; ++j) {
      if (i0 + j >= C) break;
#pragma unroll
      for (int m = 0; m < j; ++m) {
        const double2 t = cmul(lt[(i0 + m) * Cp + i0 + j], s[m]);
        s[j].x -= t.x;
        s[j].y -= t.y;
      }
      const double d = lt[(i0 + j) * Cp + i0 + j].x;
      s[j] = make_double2(s[j].x / d, s[j].y / d);
      w[(i0 + j) * 65 + lane] = s[j];
    }
  }
  __syncthreads();
  for (int i = lane; i < 64 * C; i += 64) {
    const int v = cs == 1 ? i / C : i & 63, c = cs == 1 ? i % C : i >> 6;
    const double2 u = w[c * 65 + v];
    if (k0 + v < n) x[(k0 + v) * vs + c * cs] = make_float2((float)u.x, (float)u.y);
  }
}

struct CoilLayout {
  unsigned *status = nullptr;  // the call's status word (start of the workspace)
  double2 *part = nullptr, *g = nullptr, *v = nullptr, *L = nullptr;
  int nblk = 0;
};

int layout_coils(int32_t C, int64_t T, Arena &a, CoilLayout *cl) {
  if (C < 1 || C > kMaxCoils) return fail(EXPENC_EINVAL, "ncoils must be in [1, %d] (got %d)", kMaxCoils, C);
  if (T < 0) return fail(EXPENC_EINVAL, "nsamples must be >= 0");
  cl->status = take_status(a);
  cl->nblk = (int)std::max<int64_t>(1, ceil_div(T, kGramChunk));
  cl->part = a.take<double2>((size_t)cl->nblk * C * C);
  cl->g = a.take<double2>((size_t)C * C);
  cl->v = a.take<double2>((size_t)C * C);
  cl->L = a.take<double2>((size_t)C * padded_rows(C));
  return a.ok() ? EXPENC_OK : EXPENC_EWORKSPACE;
}

// Dynamic LDS of the kernels for C coils (and nv virtual ones).
size_t cholesky_lds(int C) { return (size_t)C * (C + 1) * sizeof(double2); }
size_t whiten_lds(int C) { return (size_t)C * (65 + padded_rows(C)) * sizeof(double2); }
size_t jacobi_lds(int C) { return 2 * (size_t)C * (C + 1) * sizeof(double2); }
size_t compress_lds(int C, int nv) { return (size_t)nv * C * sizeof(double2) + (size_t)C * 65 * sizeof(float2); }

}  // namespace
}  // namespace expenc

using namespace expenc;

extern "C" size_t expenc_coil_workspace_size(int32_t ncoils, int64_t nsamples) {
  Arena a;
  CoilLayout cl;
  if (layout_coils(ncoils, nsamples, a, &cl) == EXPENC_EINVAL) return 0;
  return a.used + 256;
}

extern "C" int expenc_prewhiten(int32_t ncoils, const double *psi, int64_t nsamples, float *y, int32_t npix,
                                float *smaps, void *ws, size_t ws_bytes, void *stream) {
  if (!psi) return fail(EXPENC_EINVAL, "psi is NULL");
  if ((nsamples > 0 && !y) || (npix > 0 && !smaps) || npix < 0)
    return fail(EXPENC_EINVAL, "y or smaps is NULL for a non-empty size");
  CoilLayout cl;
  Arena a{static_cast<char *>(ws), ws_bytes, 0};
  const int st = layout_coils(ncoils, 0, a, &cl);
  if (st == EXPENC_EWORKSPACE || !ws)
    return fail(EXPENC_EWORKSPACE, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                expenc_coil_workspace_size(ncoils, 0));
  EX_TRY(st);
  hipStream_t s = (hipStream_t)stream;
  const int C = ncoils;
  const size_t clds = cholesky_lds(C), wlds = whiten_lds(C);
  EX_TRY(allow_lds(reinterpret_cast<const void *>(k_cholesky), clds, cholesky_lds(kMaxCoils)));
  EX_TRY(allow_lds(reinterpret_cast<const void *>(k_whiten), wlds, whiten_lds(kMaxCoils)));
  k_cholesky<<<1, 512, clds, s>>>(reinterpret_cast<const double2 *>(psi), C, cl.L, cl.status);
  EX_LAUNCHED("cholesky");
  if (nsamples > 0) {
    k_whiten<<<(unsigned)ceil_div(nsamples, 64), 64, wlds, s>>>(cl.L, C, reinterpret_cast<float2 *>(y), nsamples, C, 1);
    EX_LAUNCHED("whiten data");
  }
  if (npix > 0) {
    k_whiten<<<(unsigned)ceil_div(npix, 64), 64, wlds, s>>>(cl.L, C, reinterpret_cast<float2 *>(smaps), npix, 1, npix);
    EX_LAUNCHED("whiten maps");
  }
  return EXPENC_OK;
}

extern "C" int expenc_coil_compress(int32_t ncoils, int32_t nvirtual, int64_t nsamples, const float *y, int32_t npix,
                                    const float *smaps, float *y_out, float *smaps_out, double *eigvec,
                                    double *eigval, void *ws, size_t ws_bytes, void *stream) {
  if (nsamples < 1 || !y) return fail(EXPENC_EINVAL, "compression needs data (nsamples >= 1, y not NULL)");
  if (nvirtual < 1 || nvirtual > ncoils) return fail(EXPENC_EINVAL, "nvirtual must be in [1, ncoils]");
  if (npix < 0 || (npix > 0 && (!smaps || !smaps_out))) return fail(EXPENC_EINVAL, "smaps or smaps_out is NULL");
  CoilLayout cl;
  Arena a{static_cast<char *>(ws), ws_bytes, 0};
  const int st = layout_coils(ncoils, nsamples, a, &cl);
  if (st == EXPENC_EWORKSPACE || !ws)
    return fail(EXPENC_EWORKSPACE, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                expenc_coil_workspace_size(ncoils, nsamples));
  EX_TRY(st);
  hipStream_t s = (hipStream_t)stream;
  const int C = ncoils;
  const int no = C * (C + 1) / 2;
  k_gram_part<<<dim3((unsigned)cl.nblk, (unsigned)ceil_div(no, 256)), 256, (size_t)kGramChunk * C * sizeof(float2),
                s>>>(reinterpret_cast<const float2 *>(y), nsamples, C, cl.part);
  EX_LAUNCHED("gram partials");
  k_gram_sum<<<(unsigned)ceil_div(no, 64), 64, 0, s>>>(cl.part, cl.nblk, C, cl.g);
  EX_LAUNCHED("gram sum");
  double2 *v = eigvec ? reinterpret_cast<double2 *>(eigvec) : cl.v;
  const size_t jlds = jacobi_lds(C);
  EX_TRY(allow_lds(reinterpret_cast<const void *>(k_jacobi), jlds, jacobi_lds(kMaxCoils)));
  k_jacobi<<<1, kJacobiThreads, jlds, s>>>(cl.g, C, 40, v, eigval, cl.status);
  EX_LAUNCHED("jacobi");
  const size_t xlds = compress_lds(C, nvirtual);
  EX_TRY(allow_lds(reinterpret_cast<const void *>(k_compress), xlds, compress_lds(kMaxCoils, kMaxCoils)));
  if (y_out) {
    k_compress<<<(unsigned)ceil_div(nsamples, 64), 256, xlds, s>>>(v, C, nvirtual, reinterpret_cast<const float2 *>(y),
                                                                   C, 1, reinterpret_cast<float2 *>(y_out), nvirtual, 1,
                                                                   nsamples);
    EX_LAUNCHED("compress data");
  }
  if (npix > 0) {
    k_compress<<<(unsigned)ceil_div(npix, 64), 256, xlds, s>>>(v, C, nvirtual, reinterpret_cast<const float2 *>(smaps),
                                                               1, npix, reinterpret_cast<float2 *>(smaps_out), 1, npix,
                                                               npix);
    EX_LAUNCHED("compress maps");
  }
  return EXPENC_OK;
}
