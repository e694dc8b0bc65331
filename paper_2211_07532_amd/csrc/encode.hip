// Expanded encoding operator A_exp and its adjoint on gfx950.
//
// The entry of A_exp (eq. 1; the Introduction and Methods 2.1 list its
// ingredients: B0 map, spherical-harmonic field dynamics, coil maps, any
// trajectory) is
//     A[(t,c), r] = S_c(r) exp(i phi(t,r)),  phi = sum_l k_l(t) b_l(r) + dw0(r) t.
// Both operators are evaluated as complex GEMMs whose phase tile E = exp(i phi)
// is generated on the fly and never stored:
//   forward  Y[t, col] = sum_r E(t,r) Z[r, col],        Z[r, b*C+c] = S_c(r) x_b(r)
//   adjoint  X[r, col] = sum_t conj(E(t,r)) Y[t, col],  x_b(r) = sum_c conj(S_c(r)) X[r, b*C+c]
// Phase in turns: kap[t][.] = (k_l(t)/2pi, t), bet[r][.] = (b_l(r), dw0(r)/2pi);
// phi/2pi = sum_j kap[t][j] bet[r][j] is accumulated in FP64 (|phi| reaches
// tens of turns, and the sine needs ~1e-8 turn accuracy), reduced by whole turns
// (to [-1/2, 1/2] in the FP32 form and the field gradient, which then round it to
// FP32, the split forms' anchors to [0, 1)), and fed to the hardware v_sin/v_cos
// (argument in turns).
//
// The contractions are f32.hip's (FP32 form) and split.hip's / split_adj.hip's
// (bf16 and fp16 hi/lo forms); the reduction index is split across workgroups
// (split-K), and this file adds the partial sums in a fixed order, so results
// are bitwise reproducible.
#include <atomic>
#include <cmath>
#include <cstdio>
#include <limits>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "internal.h"

namespace expenc {


// ---------------------------------------------------------------------------
// Split-K reductions (fixed summation order)
// ---------------------------------------------------------------------------

// Sum of the n splits' values p[k * step], k = 0 .. n - 1, in FP64 and in k
// order, eight loads in flight per step (a loop that loads and adds one at a
// time waits for memory once per value); the last step repeats the last value.
__device__ inline void sum_strided(const float2 *__restrict__ p, int64_t step, int n, double &sx, double &sy) {
  int k = 0;
  for (; k + 8 <= n; k += 8) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(k + u) * step];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      sx += split_sign(u) * v[u].x;
      sy += split_sign(u) * v[u].y;
    }
  }
  if (k < n) {
    float2 v[7];
#pragma unroll
    for (int u = 0; u < 7; ++u) v[u] = p[min(k + u, n - 1) * step];
#pragma unroll
    for (int u = 0; u < 7; ++u)
      if (k + u < n) {
        sx += split_sign(u) * v[u].x;
        sy += split_sign(u) * v[u].y;
      }
  }
}

// scl: the scaled form's operand powers of two ([P][2]), or NULL.
__global__ void k_fwd_reduce_out(const float2 *__restrict__ part, int nsplit, int64_t T,
                                 int64_t Tp, int C, int NC, int NCP, float2 *__restrict__ y,
                                 const float *__restrict__ scl) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= T * NC) return;
  const int pz = blockIdx.y;
  part += pz * nsplit * Tp * NCP;
  y += pz * T * NC;
  int64_t t = i / NC;
  int col = (int)(i % NC);
  double sx = 0.0, sy = 0.0;
  sum_strided(part + t * NCP + col, Tp * NCP, nsplit, sx, sy);
  if (scl) {
    const double inv = 1.0 / scl[2 * pz];
    sx *= inv;
    sy *= inv;
  }
  int b = col / C, c = col % C;
  y[((int64_t)b * T + t) * C + c] = make_float2((float)sx, (float)sy);
}

// x_b(r) = alpha * sum_c conj(S_c(r)) sum_split part[split][r][b*C+c].
// Block: 8 pixels x 32 lanes; lanes stride over coils, then a shuffle sum.
__global__ __launch_bounds__(256) void k_adj_reduce_out(const float2 *__restrict__ part, int nsplit,
                                                        int R, int Rp, int nx, int C, int B, int NCP,
                                                        const float2 *__restrict__ smaps,
                                                        float2 *__restrict__ x, int64_t x_stride,
                                                        int x_row_stride, const double *__restrict__ alpha_dev,
                                                        const float2 *__restrict__ add,
                                                        const float2 *__restrict__ base, int nxq,
                                                        int64_t x_pstride, int pad_nx, int pad_ny,
                                                        const float *__restrict__ scl) {
  const int sub = threadIdx.x & 31;
  const int q = blockIdx.x * 8 + (threadIdx.x >> 5);  // pixel of x's grid
  const int npx = pad_nx > 0 ? pad_nx * pad_ny : R;
  if (q >= npx) return;  // uniform per 32-lane group
  const int pz = blockIdx.y;  // problem
  part += (int64_t)pz * nsplit * Rp * NCP;
  smaps += (int64_t)pz * C * R;
  x += pz * x_pstride;
  if (alpha_dev) alpha_dev += pz;
  if (add) add += pz * x_pstride;
  if (base) base += pz * x_pstride;
  if (pad_nx > 0) {
    // padded grid: outside the encoded nx x ny block x = add (or 0)
    const int yy = q / pad_nx, xx = q % pad_nx;
    if (yy >= R / nx || xx >= nx) {
      if (sub == 0)
        for (int b = 0; b < B; ++b) {
          const int64_t o = b * x_stride + (int64_t)yy * x_row_stride + xx;
          x[o] = add ? add[o] : make_float2(0.f, 0.f);
        }
      return;
    }
  }
  const int r = pad_nx > 0 ? (q / pad_nx) * nx + q % pad_nx : q;
  const int64_t rq = (int64_t)(r / nx) * nxq + (r % nx);  // row of the partial sums
  for (int b = 0; b < B; ++b) {
    double sx = 0.0, sy = 0.0;
    for (int c = sub; c < C; c += 32) {
      const int col = b * C + c;
      double ux = 0.0, uy = 0.0;
      sum_strided(part + rq * NCP + col, (int64_t)Rp * NCP, nsplit, ux, uy);
      float2 s = smaps[(int64_t)c * R + r];
      sx += s.x * ux + s.y * uy;  // conj(s) * u
      sy += s.x * uy - s.y * ux;
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) {
      sx += __shfl_xor(sx, o, 32);
      sy += __shfl_xor(sy, o, 32);
    }
    if (sub == 0) {
      if (scl) {
        const double inv = 1.0 / scl[2 * pz + 1];
        sx *= inv;
        sy *= inv;
      }
      const int yy = r / nx, xx = r % nx;
      const int64_t o = b * x_stride + (int64_t)yy * x_row_stride + xx;
      const double alpha = alpha_dev ? *alpha_dev : 1.0;
      if (base) {
        sx += base[o].x;
        sy += base[o].y;
      }
      float2 v = make_float2((float)(alpha * sx), (float)(alpha * sy));
      if (add) {
        v.x += add[o].x;
        v.y += add[o].y;
      }
      x[o] = v;
    }
  }
}

// Single image: x(r) = alpha * (sum over splits and ngy column blocks of the
// coil-combined partial images at row (r / nx) * nxq + r % nx), with the
// same base / add terms as k_adj_reduce_out.  Four lanes per pixel: lane j
// sums slices j, j+4, j+8, ... in order (eight loads in flight), then the
// four partial sums are added in lane order.  With pad_nx > 0 the pixels are
// those of the pad_nx x pad_ny grid, and those outside the encoded block get
// add (or 0).
__global__ __launch_bounds__(256) void k_adj_reduce_comb(const float2 *__restrict__ part, int nslice, int ngy, int Rp,
                                                         int nx, int ny, float2 *__restrict__ x, int x_row_stride,
                                                         const double *__restrict__ alpha_dev,
                                                         const float2 *__restrict__ add,
                                                         const float2 *__restrict__ base, int nxq, int64_t x_pstride,
                                                         int pad_nx, int pad_ny, const float *__restrict__ scl) {
  const int q = (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 2), j = threadIdx.x & 3;
  const int gx = pad_nx > 0 ? pad_nx : nx;
  if (q >= (pad_nx > 0 ? pad_nx * pad_ny : nx * ny)) return;  // uniform per group of four lanes
  const int pz = blockIdx.y;  // problem
  part += (int64_t)pz * nslice * Rp;
  x += pz * x_pstride;
  if (alpha_dev) alpha_dev += pz;
  if (add) add += pz * x_pstride;
  if (base) base += pz * x_pstride;
  const int yy = q / gx, xx = q % gx;
  const int64_t o = (int64_t)yy * x_row_stride + xx;
  if (yy >= ny || xx >= nx) {
    if (j == 0) x[o] = add ? add[o] : make_float2(0.f, 0.f);
    return;
  }
  const int64_t rq = (int64_t)yy * nxq + xx;
  double sx = 0.0, sy = 0.0;
  int k0 = j;
  // steps whose eight slices exist for all four lanes: unconditional loads,
  // all in flight before the first add
  for (; k0 - j + 31 < nslice; k0 += 32) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(k0 + 4 * u) * Rp + rq];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float f = split_sign((k0 + 4 * u) / ngy);
      sx += f * v[u].x;
      sy += f * v[u].y;
    }
  }
  if (k0 < nslice) {
    float2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = k0 + 4 * u < nslice ? part[(int64_t)(k0 + 4 * u) * Rp + rq] : make_float2(0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float f = split_sign((k0 + 4 * u) / ngy);
      sx += f * v[u].x;
      sy += f * v[u].y;
    }
  }
  // lane order: ((s0 + s1) + s2) + s3
  const int l0 = (threadIdx.x & 63) & ~3;
  double tx = __shfl(sx, l0), ty = __shfl(sy, l0);
#pragma unroll
  for (int u = 1; u < 4; ++u) {
    tx += __shfl(sx, l0 + u);
    ty += __shfl(sy, l0 + u);
  }
  if (j != 0) return;
  if (scl) {
    const double inv = 1.0 / scl[2 * pz + 1];
    tx *= inv;
    ty *= inv;
  }
  if (base) {
    tx += base[o].x;
    ty += base[o].y;
  }
  const double alpha = alpha_dev ? *alpha_dev : 1.0;
  float2 v = make_float2((float)(alpha * tx), (float)(alpha * ty));
  if (add) {
    v.x += add[o].x;
    v.y += add[o].y;
  }
  x[o] = v;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static int phase_terms(int L) {
  if (L + 1 <= 4) return 4;
  if (L + 1 <= 10) return 10;
  return 17;
}

constexpr int kTargetWorkgroups = 2048;
constexpr int kMaxWorkgroups = 4608;  // of the default split (scratch grows with the splits)

// EXPENC_TARGET_WG, or 0.
static int env_target() {
  static int v = [] {
    const char *e = getenv("EXPENC_TARGET_WG");
    return std::max(0, e ? atoi(e) : 0);
  }();
  return v;
}

// Chunk of the K summed indexes of a contraction of `nrb` row blocks for
// about `target` workgroups.
static int32_t target_chunk(int64_t K, int64_t nrb, int ngy, int target, int grain, int32_t cap) {
  int64_t want = ceil_div(target, nrb * ngy);
  want = std::max<int64_t>(1, std::min<int64_t>(want, K / 16));
  return (int32_t)std::min<int64_t>(round_up(ceil_div(K, want), grain), cap);
}

// Chunk without a tuned target: of the chunks up to `longest` (or that of
// kTargetWorkgroups, if it is longer) the one whose launch is shortest by
// this model, fitted to 27 sweeps (32 to 200 px, every precision, both
// kinds).  A CU takes n workgroups, `slots` at a time; a remainder of 1 or 2
// runs at 0.85 or 0.9 of the full rate, as if it were n / rate; `tail` more
// stand for the uneven end (1.5; 0.3 for the split forwards of two column
// groups, whose whole rounds of two workgroups end together).  A workgroup has a prologue of about 8 steps of
// 16 indexes, and a step takes 0.5 us of a CU (0.6 for the general-basis and
// 1 for the FP32 kernels, 0.6 times that with 16 columns per wave).  The
// partial sums cost `width` complex values per row and split at 8 TB/s.
// Sums longer than those of kTargetWorkgroups take `fold` times as long: they
// are the ones added up outside the matrix instruction (fwd_fold), or their
// error would grow by up to 30 % (fp16; carried through the instruction it is
// rounded at its size 6 or 12 times a step).
// Whole calls, at 2048 workgroups and as picked (folded): 100 x 90, T 3000, 16
// coils, 4 images, fp16: forward 102 / 85 us (21 splits), adjoint 99 / 88 (9);
// 64 x 64, T 4000, 8 coils, bf16: 39 / 32 and 72 / 30, FP32 49 / 47 and 55 / 54;
// 148 x 148, 32 coils, bf16 351 / 349 us (unfolded with 16 splits 335, at an error
// 0.8 % larger).
int32_t default_chunk(int64_t K, int64_t nrb, int ngy, int64_t width, int slots, double step, double tail, double fold,
                      int grain, int32_t longest, int32_t cap) {
  const int32_t at_target = target_chunk(K, nrb, ngy, kTargetWorkgroups, grain, cap);
  const int64_t last = std::max<int64_t>(at_target, std::min<int64_t>(longest, round_up(K, grain)));
  const int64_t most = std::max<int64_t>(1, kMaxWorkgroups / (nrb * ngy));
  int32_t best = at_target;
  int64_t prev = -1;
  double cost = 1e300;
  for (int64_t chunk = std::min<int64_t>(at_target, round_up(ceil_div(K, most), grain)); chunk <= last;
       chunk += grain) {
    const int64_t split = ceil_div(K, chunk);
    if (split == prev) continue;  // (the shortest chunk of a split is its most even)
    prev = split;
    const int64_t n = ceil_div(nrb * ngy * split, 256), r = n % slots;
    const double load = (double)(n - r) + (r == 1 ? 1 / 0.85 : r == 2 ? 2 / 0.9 : (double)r) + tail;
    const double t = load * (double)(chunk / 16 + 8) * step * (chunk > at_target ? fold : 1.0) +
                     (double)split * nrb * width * (256 * 8 / 8e6);
    if (t < cost) {
      cost = t;
      best = (int32_t)chunk;
    }
  }
  return best;
}

// Workgroup targets per operator geometry, batch and precision, set by the
// autotuner through expenc_set_tuning.  Plans made after a change differ, so
// the generation counter is part of every graph-cache key.
struct TuneEntry {
  int32_t nx, ny, ncoils, nbasis, basis_kind, batch, precision;
  int64_t nsamples;
  int32_t fwd_target, adj_target, col_groups;
};
static std::mutex g_tune_mu;
static std::vector<TuneEntry> g_tune;
static std::atomic<uint64_t> g_tune_gen{0};

uint64_t tuning_generation() { return g_tune_gen.load(); }

static bool tune_match(const TuneEntry &e, const expenc_op *op, int32_t batch, int32_t precision) {
  return e.nx == op->nx && e.ny == op->ny && e.ncoils == op->ncoils && e.nbasis == op->nbasis &&
         e.basis_kind == op->basis_kind && e.batch == batch && e.precision == precision &&
         e.nsamples == op->nsamples;
}

static void tuned_targets(const expenc_op *op, int32_t batch, int32_t precision, int *fwd, int *adj, int *gw) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  for (const TuneEntry &e : g_tune)
    if (tune_match(e, op, batch, precision)) {
      if (e.fwd_target > 0) *fwd = e.fwd_target;
      if (e.adj_target > 0) *adj = e.adj_target;
      if (e.col_groups > 0) *gw = e.col_groups;
      return;
    }
}

int set_tuning(const expenc_op *op, int32_t batch, int32_t precision, int32_t fwd_target, int32_t adj_target,
               int32_t col_groups) {
  if (!op) return fail(EXPENC_EINVAL, "operator descriptor is NULL");
  if (fwd_target < 0 || adj_target < 0 || fwd_target > (1 << 20) || adj_target > (1 << 20))
    return fail(EXPENC_EINVAL, "workgroup targets must be in [0, 2^20]");
  if (col_groups < 0 || col_groups > 2) return fail(EXPENC_EINVAL, "col_groups must be 0, 1 or 2");
  std::lock_guard<std::mutex> lk(g_tune_mu);
  for (size_t i = 0; i < g_tune.size(); ++i)
    if (tune_match(g_tune[i], op, batch, precision)) {
      g_tune.erase(g_tune.begin() + i);
      break;
    }
  if (fwd_target > 0 || adj_target > 0 || col_groups > 0)
    g_tune.push_back(TuneEntry{op->nx, op->ny, op->ncoils, op->nbasis, op->basis_kind, batch, precision,
                               op->nsamples, fwd_target, adj_target, col_groups});
  g_tune_gen.fetch_add(1);
  return EXPENC_OK;
}

// Pixels per step of the forward contraction (general-basis split form: 32).
static int fwd_grain(const EncPlan &q) { return q.sh || q.prec == EXPENC_FP32 ? 16 : 32; }

int make_plan(const expenc_op *op, int32_t batch, int32_t precision, EncPlan *p, int32_t nprob) {
  if (!op) return fail(EXPENC_EINVAL, "operator descriptor is NULL");
  if (op->nx < 1 || op->ny < 1) return fail(EXPENC_EINVAL, "image grid %dx%d is empty", op->nx, op->ny);
  if ((int64_t)op->nx * op->ny > (1 << 26)) return fail(EXPENC_EINVAL, "image grid too large");
  if (op->ncoils < 1) return fail(EXPENC_EINVAL, "ncoils must be >= 1 (got %d)", op->ncoils);
  if (op->nbasis < 0 || op->nbasis > 16) return fail(EXPENC_EINVAL, "nbasis must be in [0,16] (got %d)", op->nbasis);
  if (op->nsamples < 1 || op->nsamples > (int64_t(1) << 31)) return fail(EXPENC_EINVAL, "nsamples out of range");
  if (op->basis_kind != EXPENC_BASIS_MAPS && op->basis_kind != EXPENC_BASIS_SH)
    return fail(EXPENC_EINVAL, "unknown basis_kind %d", op->basis_kind);
  if (op->reserved != 0) return fail(EXPENC_EINVAL, "reserved field must be 0");
  if (op->basis_kind == EXPENC_BASIS_SH && !(op->fov_x > 0 && op->fov_y > 0))
    return fail(EXPENC_EINVAL, "EXPENC_BASIS_SH needs fov_x, fov_y > 0");
  if (op->nbasis > 0 && !op->coef) return fail(EXPENC_EINVAL, "coef NULL with nbasis > 0");
  if (op->nbasis > 0 && op->basis_kind == EXPENC_BASIS_MAPS && !op->basis)
    return fail(EXPENC_EINVAL, "basis NULL with nbasis > 0 and EXPENC_BASIS_MAPS");
  if (!op->time) return fail(EXPENC_EINVAL, "time array is NULL");
  if (!op->smaps) return fail(EXPENC_EINVAL, "smaps is NULL");
  if (batch < 1) return fail(EXPENC_EINVAL, "batch must be >= 1 (got %d)", batch);
  if (nprob < 1 || nprob > 65535) return fail(EXPENC_EINVAL, "problem count %d out of range", nprob);
  if (precision != EXPENC_FP32 && precision != EXPENC_BF16_SPLIT && precision != EXPENC_FP16_SPLIT)
    return fail(EXPENC_EINVAL, "unknown precision %d", precision);
  if ((int64_t)op->ncoils * batch > 4096) return fail(EXPENC_EUNSUPPORTED, "ncoils*batch > 4096");
  EncPlan q;
  q.nx = op->nx;
  q.ny = op->ny;
  q.R = op->nx * op->ny;
  q.sh = op->basis_kind == EXPENC_BASIS_SH;
  q.nxq = q.sh ? (int32_t)round_up(op->nx, 16) : op->nx;
  q.dx = q.sh ? op->fov_x / op->nx : 0.0;
  q.dy = q.sh ? op->fov_y / op->ny : 0.0;
  q.z0 = q.sh ? op->z0 : 0.0;
  q.Rp = (int32_t)round_up((int64_t)q.nxq * op->ny, 256);
  q.T = op->nsamples;
  q.Tp = round_up(q.T, 256);
  q.C = op->ncoils;
  q.B = batch;
  q.NC = q.C * q.B;
  q.G = (int32_t)ceil_div(q.NC, 16);
  int tgt_fwd = env_target(), tgt_adj = tgt_fwd, tuned_gw = 0;  // 0: default_chunk
  tuned_targets(op, batch, precision, &tgt_fwd, &tgt_adj, &tuned_gw);
  // 16-column groups per wave: two (one phase tile feeds both) unless tuned
  // to one or there is only one
  q.GW = (q.G >= 2 && tuned_gw != 1) ? 2 : 1;
  q.NGY = (int32_t)ceil_div(q.G, q.GW);
  q.comb = (batch == 1 && precision != EXPENC_FP32);
  q.NCP = q.NGY * q.GW * 16;  // every wave's column groups exist (zero-filled past NC)
  q.L = op->nbasis;
  q.NT = phase_terms(q.L);
  q.prec = precision;
  q.P = nprob;
  q.scaled = precision != EXPENC_BF16_SPLIT;
  // Partial sums of the default splits, unless kTargetWorkgroups makes them
  // longer: at most 64 indexes in the FP32 form, whose error they set (folded, 64
  // x 64 with 64: 0.7 of the FP32 instruction's with its 32), 1024 in the split
  // forms (below), 512 where those are not folded.
  const bool f32 = precision == EXPENC_FP32;
  const int32_t longest = f32 ? kF32FoldMax : kSplitAdjChunkMax;
  // Sums longer than those of kTargetWorkgroups are folded (see default_chunk),
  // unless a tuned target asks for them; the general-basis split forward's are
  // not: the order of its phase product leaves it 0.4 to 0.9 of the error that
  // the phases' vector arithmetic had.
  const bool fwd_folds = q.sh || f32;
  const double fold = 1.08;
  auto folds = [&](int32_t chunk, int64_t K, int64_t nrb, int tuned, int grain, int32_t cap) {
    return !tuned && chunk > target_chunk(K, nrb, q.NGY, kTargetWorkgroups, grain, cap);
  };
  const double step = (f32 ? 1.0 : q.sh ? 0.5 : 0.6) * (q.GW == 2 ? 1.0 : 0.6);
  // forward: 256 sample rows per workgroup, split over pixels
  {
    const int64_t nrb = q.Tp / 256 * q.P;
    const int32_t cap = f32 ? kF32ChunkMax : std::numeric_limits<int32_t>::max();
    const int slots = f32 ? 5 - q.GW : q.sh ? 4 - q.GW : 2;  // workgroups that fit on a CU
    const int grain = fwd_grain(q);
    q.fwd_chunk = tgt_fwd ? target_chunk(q.Rp, nrb, q.NGY, tgt_fwd, grain, cap)
                          : default_chunk(q.Rp, nrb, q.NGY, q.NCP, slots, step, f32 || q.GW == 1 ? 1.5 : 0.3,
                                          fwd_folds ? fold : 1.0, grain, fwd_folds ? longest : 512, cap);
    q.fwd_split = (int32_t)ceil_div(q.Rp, q.fwd_chunk);
    q.nwmax = (int32_t)split_grid(q.Tp / 256 * q.fwd_split) * q.NGY * 4;
    q.fwd_fold = fwd_folds && folds(q.fwd_chunk, q.Rp, nrb, tgt_fwd, grain, cap);
  }
  // adjoint: 256 pixel rows per workgroup, split over samples
  {
    const int64_t nrb = q.Rp / 256 * q.P;
    // (the split adjoints step over 32 samples at a time)
    const int grain = f32 ? 16 : 32;
    // The error of a contraction grows with the length of the sums one
    // workgroup accumulates on the matrix cores.  Measured on a 200 px,
    // T = 20000 fp16 solve: NRMSE 1.8e-5 at 562 samples per split adjoint
    // chunk, 2.9e-5 at 5056, 5.0e-5 at 10112 (the split forward's chunk
    // length did not matter); with 12 problems per launch the FP32 anchors'
    // chunks (3 forward, 2 adjoint splits) alone took it from 2.2e-5 to
    // 4.9e-5.  So chunks are capped (the tuned single-problem shapes are
    // below the caps).
    const int32_t cap = f32 ? kF32ChunkMax : kSplitAdjChunkMax;
    const int slots = f32 ? 5 - q.GW : q.sh ? 3 : 2;
    q.adj_chunk = tgt_adj ? target_chunk(q.Tp, nrb, q.NGY, tgt_adj, grain, cap)
                          : default_chunk(q.Tp, nrb, q.NGY, q.comb ? q.NGY : q.NCP, slots, step, 1.5, fold, grain,
                                          std::min(longest, cap), cap);
    q.adj_split = (int32_t)ceil_div(q.Tp, q.adj_chunk);
    q.adj_fold = folds(q.adj_chunk, q.Tp, nrb, tgt_adj, grain, cap);
  }
  *p = q;
  return EXPENC_OK;
}

static size_t enc_bytes(const EncPlan &p, int need) {
  Arena a;
  EncBuffers b;
  carve_enc(p, a, &b, need);
  return a.used + 256;
}

// (one size for both directions: a caller may keep one workspace for them)
size_t enc_operand_bytes(const EncPlan &p) { return std::max(enc_bytes(p, kNeedForward), enc_bytes(p, kNeedAdjoint)); }

int plan_forward_within(const expenc_op *op, int32_t batch, int32_t precision, size_t cap, EncPlan *p) {
  EncPlan q;
  EX_TRY(make_plan(op, batch, precision, &q));
  const int32_t min_split = q.prec == EXPENC_FP32 ? (int32_t)ceil_div(q.Rp, kF32ChunkMax) : 1;
  auto set_split = [&](int32_t want) {
    q.fwd_chunk = (int32_t)round_up(ceil_div(q.Rp, want), fwd_grain(q));
    if (q.prec == EXPENC_FP32) q.fwd_chunk = std::min(q.fwd_chunk, kF32ChunkMax);
    q.fwd_split = (int32_t)ceil_div(q.Rp, q.fwd_chunk);
    q.nwmax = (int32_t)split_grid(q.Tp / 256 * q.fwd_split) * q.NGY * 4;
    q.fwd_fold = q.sh || q.prec == EXPENC_FP32;
  };
  auto fits = [&] { return enc_bytes(q, kNeedForward) <= cap; };
  while (!fits() && q.fwd_split > min_split)
    set_split(std::max<int32_t>(min_split, q.fwd_split - std::max<int32_t>(1, q.fwd_split / 4)));
  // the FP32 form's records take three times the operand's bytes: hold those of
  // fewer splits, then of fewer column blocks (whose phases are evaluated again)
  if (q.prec == EXPENC_FP32 && !fits()) {
    q.pass_split = q.fwd_split;
    q.pass_gy = q.NGY;
    while (!fits() && q.pass_split > 1) q.pass_split = (q.pass_split + 1) / 2;
    while (!fits() && q.pass_gy > 1) q.pass_gy = (q.pass_gy + 1) / 2;
  }
  if (!fits())
    return fail(EXPENC_EWORKSPACE, "the forward of this operator needs %zu bytes of scratch, more than the %zu "
                "of the static scratch (use expenc_forward with a workspace)", enc_bytes(q, kNeedForward), cap);
  *p = q;
  return EXPENC_OK;
}

int carve_enc(const EncPlan &p, Arena &a, EncBuffers *b, int need, std::initializer_list<const EncPlan *> with) {
  const bool fwd = (need & kNeedForward) != 0, adj = (need & kNeedAdjoint) != 0;
  const size_t P = p.P;
  size_t part = 0, rec = 0, yop = 0;
  int32_t nwmax = 0;
  bool scaled = false, f32 = false;
  auto plan = [&](const EncPlan &q) {
    const size_t g = q.NCP / 16 * (q.prec == EXPENC_FP32 ? 384 : 256);  // record bytes per index
    if (fwd) {
      part = std::max(part, P * q.fwd_split * q.Tp * q.NCP);
      rec = std::max(rec, q.pass_split ? (size_t)std::min<int64_t>(q.Rp, (int64_t)q.pass_split * q.fwd_chunk) *
                                             std::min(q.NCP / 16, q.pass_gy * q.GW) * 384
                                       : P * q.Rp * g);
      nwmax = std::max(nwmax, q.nwmax);
    }
    if (adj) {
      part = std::max(part, P * q.adj_split * q.Rp * (q.comb ? q.NGY : q.NCP));
      rec = std::max(rec, P * q.Tp * g);
    }
    if (q.prec == EXPENC_FP32) {
      f32 = true;
      if (need == kNeedBoth) yop = std::max(yop, P * q.Tp * q.NCP);
    }
    scaled = scaled || q.scaled;
  };
  plan(p);
  for (const EncPlan *q : with) plan(*q);
  b->part = a.take<float2>(part);
  b->zs = b->ys = a.take<char>(rec);
  if (yop) b->yop = a.take<float2>(yop);
  const bool split = p.prec != EXPENC_FP32;
  if (p.sh) {
    // polynomial phase tables
    if (fwd || f32) b->pmono = a.take<double>(P * p.Tp * kPolyStride);
    b->dwq = a.take<double>(P * p.Rp);
    if (split && fwd) b->ddw = a.take<float>(P * p.Rp);
    if (split && adj) {
      b->dpa = a.take<float>(P * p.Tp * 16);
      b->anc = a.take<float>(P * (p.Tp / 32) * p.Rp);
    }
  } else {
    b->kap = a.take<double>(P * p.Tp * p.NT);
    b->bet = a.take<double>(P * p.Rp * p.NT);
    if (split && fwd) b->dbet = a.take<float>(P * p.Rp * round_up(p.NT, 2));
    if (split && adj) b->dkap = a.take<float>(P * p.Tp * round_up(p.NT, 2));
  }
  if (p.comb && adj) b->sq = a.take<float2>(P * p.Rp * p.NCP);
  if (scaled) {
    b->scl = a.take<float>(P * 2);
    b->amax = a.take<float>(P * 3 * kAmaxBlocks);
    b->wmax = a.take<float>(std::max<size_t>(1, P * nwmax));
  }
  return a.ok() ? EXPENC_OK : EXPENC_EWORKSPACE;
}

static inline dim3 grid_p(int64_t n, int bs, int P) { return dim3((unsigned)ceil_div(n, bs), (unsigned)P); }

int enc_build_z(const EncPlan &p, const float *smaps, const float2 *x, int64_t x_stride,
                int32_t x_row_stride, const EncBuffers &b, hipStream_t s, const float2 *xsub, int64_t x_pstride,
                bool prepared) {
  if (prepared && !p.scaled) return EXPENC_OK;  // enc_prepare wrote the records
  if (p.prec != EXPENC_FP32)
    return split_build_z(p, smaps, x, xsub, x_stride, x_row_stride, b, s, x_pstride, prepared);
  if (xsub) return fail(EXPENC_EUNSUPPORTED, "operand difference is only built for split forms");
  return f32_build_z(p, smaps, x, x_stride, x_row_stride, b, s, x_pstride, prepared);
}

int enc_pack_y(const EncPlan &p, const float2 *y, const EncBuffers &b, hipStream_t s, float sign, bool prepared) {
  if (prepared && !p.scaled) return EXPENC_OK;
  if (p.prec != EXPENC_FP32) {
    if (sign != 1.f) return fail(EXPENC_EUNSUPPORTED, "scaled operand packing is FP32 only");
    return split_pack_y(p, y, false, nullptr, b, s, prepared);
  }
  return f32_pack_y(p, y, sign, nullptr, b, s, prepared);
}

// ---------------------------------------------------------------------------
// Opt-in per-kernel timing of the two contraction kernels with HIP events
// recorded on the launch stream (eager launches only; skipped while the
// stream is being captured into a graph).
// ---------------------------------------------------------------------------
namespace {
struct KernelTimer {
  std::mutex mu;
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[2];
  std::vector<hipEvent_t> pool;
  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    hipEventCreate(&e);
    return e;
  }
  void clear() {
    for (auto &v : ev)
      for (auto &pr : v) {
        pool.push_back(pr.first);
        pool.push_back(pr.second);
      }
    ev[0].clear();
    ev[1].clear();
  }
};
KernelTimer g_timer;

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) return true;
  return st != hipStreamCaptureStatusNone;
}

template <class F>
void timed(int kind, hipStream_t s, F launch) {
  hipEvent_t a = nullptr, b = nullptr;
  bool t = false;
  {
    std::lock_guard<std::mutex> lk(g_timer.mu);
    t = g_timer.on && !capturing(s);
    if (t) {
      a = g_timer.get();
      b = g_timer.get();
    }
  }
  if (t) hipEventRecord(a, s);
  launch();
  if (t) {
    hipEventRecord(b, s);
    std::lock_guard<std::mutex> lk(g_timer.mu);
    g_timer.ev[kind].push_back({a, b});
  }
}
}  // namespace

int kernel_timing(int32_t mode, double *out) {
  std::lock_guard<std::mutex> lk(g_timer.mu);
  if (mode == 0 || mode == 1) {
    g_timer.clear();
    g_timer.on = (mode == 1);
    return EXPENC_OK;
  }
  if (mode != 2 || !out) return fail(EXPENC_EINVAL, "bad timing mode");
  for (int k = 0; k < 2; ++k) {
    double tot = 0;
    for (auto &pr : g_timer.ev[k]) {
      EX_HIP(hipEventSynchronize(pr.second));
      float ms = 0;
      EX_HIP(hipEventElapsedTime(&ms, pr.first, pr.second));
      tot += ms;
    }
    out[2 * k] = tot;
    out[2 * k + 1] = (double)g_timer.ev[k].size();
  }
  return EXPENC_OK;
}

int enc_forward_partials(const EncPlan &p, const EncBuffers &b, hipStream_t s, bool timing) {
  auto launch = [&] {
    if (p.prec != EXPENC_FP32) {
      split_forward_launch(p, b, s);
      return;
    }
    f32_forward_launch(p, b, s);
  };
  if (timing) timed(0, s, launch);
  else launch();
  EX_LAUNCHED("forward contraction");
  return EXPENC_OK;
}

int enc_adjoint_partials(const EncPlan &p, const EncBuffers &b, hipStream_t s) {
  if (p.comb && !b.sq) return fail(EXPENC_EINVAL, "coil table of a single-image split plan is not carved");
  if (p.sh && p.prec != EXPENC_FP32 && !b.anc) return fail(EXPENC_EINVAL, "anchor table of a split plan is not carved");
  int st = EXPENC_OK;
  timed(1, s, [&] {
    if (p.prec != EXPENC_FP32) {
      split_adjoint_launch(p, b, s);
      return;
    }
    st = f32_adjoint_launch(p, b, s);
  });
  EX_TRY(st);
  EX_LAUNCHED("adjoint contraction");
  return EXPENC_OK;
}

int enc_forward_reduce_out(const EncPlan &p, const EncBuffers &b, float2 *y, hipStream_t s) {
  k_fwd_reduce_out<<<grid_p(p.T * p.NC, 256, p.P), 256, 0, s>>>(b.part, p.fwd_split, p.T, p.Tp, p.C, p.NC, p.NCP, y,
                                                                  p.scaled ? b.scl : nullptr);
  EX_LAUNCHED("forward reduce");
  return EXPENC_OK;
}

int enc_forward_residual(const EncPlan &p, const EncBuffers &b, const float2 *y_meas, hipStream_t s, bool *y_bounded) {
  if (p.prec != EXPENC_FP32) return split_pack_y(p, nullptr, true, y_meas, b, s, false, y_bounded);
  return f32_pack_y(p, nullptr, 1.f, y_meas, b, s, false, y_bounded);
}

int enc_adjoint_reduce_out(const EncPlan &p, const EncBuffers &b, const float *smaps, float2 *x,
                           int64_t x_stride, int32_t x_row_stride, const double *alpha_dev,
                           const float2 *add, hipStream_t s, const float2 *base, int64_t x_pstride,
                           int32_t pad_nx, int32_t pad_ny) {
  const int64_t npx = pad_nx > 0 ? (int64_t)pad_nx * pad_ny : p.R;
  if (pad_nx > 0 && (pad_nx < p.nx || pad_ny < p.ny || x_row_stride < pad_nx))
    return fail(EXPENC_EINVAL, "padded grid %dx%d smaller than the image", pad_nx, pad_ny);
  if (p.comb) {
    k_adj_reduce_comb<<<grid_p(npx * 4, 256, p.P), 256, 0, s>>>(b.part, p.adj_split * p.NGY, p.NGY, p.Rp, p.nx, p.ny, x,
                                                          x_row_stride, alpha_dev, add, base, p.nxq, x_pstride,
                                                          pad_nx, pad_ny, p.scaled ? b.scl : nullptr);
    EX_LAUNCHED("adjoint reduce");
    return EXPENC_OK;
  }
  k_adj_reduce_out<<<grid_p(npx, 8, p.P), 256, 0, s>>>(b.part, p.adj_split, p.R, p.Rp, p.nx, p.C, p.B, p.NCP,
                                                       reinterpret_cast<const float2 *>(smaps), x, x_stride,
                                                       x_row_stride, alpha_dev, add, base, p.nxq, x_pstride,
                                                       pad_nx, pad_ny, p.scaled ? b.scl : nullptr);
  EX_LAUNCHED("adjoint reduce");
  return EXPENC_OK;
}

}  // namespace expenc
