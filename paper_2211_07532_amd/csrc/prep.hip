// Field setup of the encoding operators: the phase tables of both basis
// kinds, the coil table of the split adjoint's epilogue, and of a single
// application's operand the records (bf16) or the magnitude bounds (FP32, fp16),
// all in ONE launch whose workgroups take one role each (a range of block
// indices per table).  No table reads another: where
// one is built from a second (increments and anchors from the polynomial
// coefficients), its workgroup evaluates that again from the inputs.  A call
// that applies one direction only prepares what that direction reads.
//
// Bound: the anchor table's stores ([Tp/32][Rp] floats; 65 MB at 170 x 170,
// T = 17340) and, for small problems, launches.  For one fp16 adjoint of that
// size with 20 coils: 28 us, where eight kernels took 130 us (62 of them the
// anchors, one entry per thread with two index divisions and its own
// coefficient loads; 22 the polynomial coefficients, whose per-thread arrays
// were indexed at run time; 12 a bound of the coil maps only a forward reads).
// The bf16 records here instead of in a launch of their own: 33 x 20, 17 coils
// 24.5 -> 21.2 us.  The scaled forms' records need the bound first: a launch of
// their own (32 x 32, 8 coils, FP32 forward 25.6 us; records here, every
// workgroup bounding the whole operand itself, 26.8; unscaled records here,
// which lose the operands' last bits below 2^-110, 21.7).
#include "internal.h"
#include "split_dev.h"

namespace expenc {

static constexpr double kInv2Pi = 0.15915494309189533576888376337251436;
constexpr int kAncTiles = 16;  // 32-sample tiles per anchor workgroup

enum PrepRole { kRoleAnchor, kRoleRecords, kRolePoly, kRoleIncr, kRolePixel, kRoleSq, kRoleKap, kRoleBet, kRoleMaps,
                kRoleOperand, kRoles };

struct PrepArgs {
  const double *coef, *time, *basis, *dw0, *z0s;
  const float2 *smaps, *operand;
  double *kap, *bet, *pmono, *dwq;
  float *dkap, *dbet, *ddw, *dpa, *anc, *amax;
  float2 *sq;
  int64_t T, Tp, nop;  // nop: operand elements per problem
  int R, Rp, L, NT, nx, ny, nxq, C, NC, NCP, op_l1;
  u32x4 *rec;
  int rec_image, rec_perm, rec_chunk;  // records of an image; index order; indexes per split
  double dx, dy, z0;
  unsigned end[kRoles];  // block index one past each role's range
};

// The ten monomial coefficients (turns; order 1, x, y, x^2, xy, y^2, x^3,
// x^2 y, x y^2, y^3) of sum_l k_l(t) b_l(x, y, z) at fixed z, and t: the
// solid harmonics multiplied out, terms added in the order of l.  Padding repeats
// the last sample, here and in every table (pixels: the last of their row and
// the last row): a tile's centre, whose phase the FP32 differences within the tile start
// from, may be padding.
__device__ inline void sample_poly(const double *__restrict__ coef, const double *__restrict__ time, int64_t t,
                                   int64_t T, int L, double z, double (&P)[11]) {
  t = min(t, T - 1);
  const double *c = coef + t * L;
  double k[16];
#pragma unroll
  for (int l = 0; l < 16; ++l) k[l] = l < L ? c[l] * kInv2Pi : 0.0;
  const double z2 = z * z;
  P[0] = fma(k[12], 2 * z2 * z, fma(k[6], 2 * z2, fma(k[3], z, k[0])));
  P[1] = fma(k[13], 4 * z2, fma(k[7], z, k[1]));
  P[2] = fma(k[11], 4 * z2, fma(k[5], z, k[2]));
  P[3] = fma(k[14], z, fma(k[12], -3 * z, k[8] - k[6]));
  P[4] = fma(k[10], z, k[4]);
  P[5] = fma(k[14], -z, fma(k[12], -3 * z, -k[6] - k[8]));
  P[6] = k[15] - k[13];
  P[7] = fma(k[9], 3.0, -k[11]);
  P[8] = fma(k[15], -3.0, -k[13]);
  P[9] = -k[9] - k[11];
  P[10] = time[t];
}

// dw0/2pi at padded pixel rq
__device__ inline double pixel_dw(const double *__restrict__ dw0, int rq, int nx, int ny, int nxq) {
  const int yy = rq / nxq, xx = rq - yy * nxq;
  return dw0 ? dw0[(int64_t)min(yy, ny - 1) * nx + min(xx, nx - 1)] * kInv2Pi : 0.0;
}

// Element (index i, term j) of a difference table of the split contractions:
// per 32 indexes [pair of terms][term of the pair][index], zero past NT.
__device__ inline void put_diff(float *__restrict__ d, int64_t i, int j, int NT, float v) {
  float *o = d + ((i >> 5) * ((NT + 1) / 2) + (j >> 1)) * 64 + (i & 31);
  o[32 * (j & 1)] = v;
  if ((NT & 1) && j == NT - 1) o[32] = 0.f;
}

__global__ __launch_bounds__(256) void k_prepare(PrepArgs a) {
  __shared__ double pc[kAncTiles][12];
  __shared__ float wm[4];
  const int64_t pz = blockIdx.y;  // problem
  int role = 0;
  while (blockIdx.x >= a.end[role]) ++role;
  const unsigned blk = blockIdx.x - (role ? a.end[role - 1] : 0u);
  const int tid = threadIdx.x;
  const int nte = (a.NT + 1) & ~1;
  const int64_t i = (int64_t)blk * 256 + tid;
  const double z = a.z0s ? a.z0s[pz] : a.z0;
  const double *coef = a.coef ? a.coef + pz * a.T * a.L : nullptr;
  const double *time = a.time + pz * a.T;
  const double *dw0 = a.dw0 ? a.dw0 + pz * a.R : nullptr;
  if (role == kRoleAnchor) {
    // phase of each 32-sample tile's centre sample at each pixel, in FP64
    // (nested in y, then in x), reduced to turns in [0, 1): 256 pixels x
    // kAncTiles tiles per workgroup, the tiles' coefficients in LDS
    const int npb = a.Rp / 256;
    const int64_t q0 = (int64_t)(blk / npb) * kAncTiles;
    const int rq = (int)(blk % npb) * 256 + tid;
    const int64_t nq = a.Tp / 32;
    if (tid < kAncTiles) {
      double P[11];
      sample_poly(coef, time, 32 * (q0 + tid) + 16, a.T, a.L, z, P);
#pragma unroll
      for (int m = 0; m < 11; ++m) pc[tid][m] = P[m];
    }
    __syncthreads();
    const int yy = rq / a.nxq;
    const double x = (rq - yy * a.nxq - 0.5 * a.nx) * a.dx, y = (yy - 0.5 * a.ny) * a.dy;
    const double w = pixel_dw(dw0, rq, a.nx, a.ny, a.nxq);
    float *out = a.anc + pz * nq * a.Rp + rq;
    for (int j = 0; j < kAncTiles && q0 + j < nq; ++j) {
      const double *p = pc[j];
      const double a0 = fma(y, fma(y, fma(y, p[9], p[5]), p[2]), p[0]);
      const double a1 = fma(y, fma(y, p[8], p[4]), p[1]);
      const double a2 = fma(y, p[7], p[3]);
      out[(q0 + j) * a.Rp] = (float)__builtin_amdgcn_fract(fma(p[10], w, fma(x, fma(x, fma(x, p[6], a2), a1), a0)));
    }
    return;
  }
  if (role == kRoleRecords) {
    // operand records from the call's image (times the coil maps) or data, as
    // the packing kernels write them; every load before the first use
    const int NGP = a.NCP / 16;
    const int64_t K = a.rec_image ? a.Rp : a.Tp;
    if (i >= K / 16 * NGP * 64) return;
    const int lane = (int)(i & 63), hl = lane >> 5, im = (lane >> 4) & 1;
    const int64_t qg = i >> 6, k0 = qg / NGP * 16;
    const int g = (int)(qg % NGP), col = 16 * g + (lane & 15);
    const bool colok = col < a.NC;
    const int b = colok ? col / a.C : 0, c = colok ? col % a.C : 0;
    const float2 *op = a.operand + pz * a.nop, *sm = a.smaps + (pz * a.C + c) * a.R;
    float2 v[8], sv[8];
    bool ok[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t k = k0 + (a.rec_perm ? 8 * (e >> 2) + 4 * hl + (e & 3) : 8 * hl + e);
      if (a.rec_image) {
        const int yy = (int)k / a.nxq, xx = (int)k - yy * a.nxq;
        ok[e] = colok && xx < a.nx && yy < a.ny;
        const int64_t o = ok[e] ? (int64_t)yy * a.nx + xx : 0;
        v[e] = op[(int64_t)b * a.R + o];
        sv[e] = sm[o];
      } else {
        ok[e] = colok && k < a.T;
        v[e] = op[((int64_t)b * a.T + (ok[e] ? k : 0)) * a.C + c];
        sv[e] = make_float2(0.f, 0.f);
      }
    }
    const float f = split_sign(k0 / a.rec_chunk);
    float b1[8], b2[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float2 z = v[e];
      if (a.rec_image)
        z = make_float2(sv[e].x * v[e].x - sv[e].y * v[e].y, sv[e].x * v[e].y + sv[e].y * v[e].x);
      z = ok[e] ? make_float2(z.x * f, z.y * f) : make_float2(0.f, 0.f);
      b1[e] = im ? z.y : z.x;
      b2[e] = im ? z.x : z.y;
      if (im != a.rec_image) b2[e] = -b2[e];
    }
    write_record<true>(a.rec + pz * K * NGP * 16, qg / NGP, g, NGP, lane, b1, b2);
    return;
  }
  if (role == kRolePoly) {
    if (i >= a.Tp) return;
    double P[11];
    sample_poly(coef, time, i, a.T, a.L, z, P);
    double *o = a.pmono + (pz * a.Tp + i) * kPolyStride;
#pragma unroll
    for (int m = 0; m < 11; ++m) o[m] = P[m];
    return;
  }
  if (role == kRoleIncr) {
    // A operand of the adjoint's phase-increment product, in lane order.  For
    // the 32-sample tile q and lane l (sample t = 32q + l%32, half hl = l/32),
    // with d_m the coefficients of t minus those of the centre 32q + 16, the
    // increment at a pixel of image row y is the cubic in x
    //   C_0 + C_1 x + C_2 x^2 + C_3 x^3 + d10 dw0,
    //   C_0 = d0 + d2 y + d5 y^2 + d9 y^3,  C_1 = d1 + d4 y + d8 y^2,
    //   C_2 = d3 + d7 y,                    C_3 = d6,
    // and lane l holds the coefficients the adjoint evaluates at a block's
    // row: [0..3] the cubic in y of C_hl, [4..5] the linear one of C_{2+hl},
    // [6] d10 (hl = 0, the dw0 term) or 1 (hl = 1, the anchor term).
    if (i >= a.Tp * 2) return;
    const int64_t q = i >> 6;
    const int l = (int)(i & 63);
    double d[11], e[11];
    sample_poly(coef, time, 32 * q + (l & 31), a.T, a.L, z, d);
    sample_poly(coef, time, 32 * q + 16, a.T, a.L, z, e);
#pragma unroll
    for (int m = 0; m < 11; ++m) d[m] -= e[m];
    const bool hl = (l >> 5) != 0;
    float4 *o = reinterpret_cast<float4 *>(a.dpa + (pz * a.Tp * 2 + i) * 8);
    o[0] = make_float4((float)(hl ? d[1] : d[0]), (float)(hl ? d[4] : d[2]), (float)(hl ? d[8] : d[5]),
                       (float)(hl ? 0.0 : d[9]));
    o[1] = make_float4((float)(hl ? d[6] : d[3]), (float)(hl ? 0.0 : d[7]), (float)(hl ? 1.0 : d[10]), 0.f);
    return;
  }
  if (role == kRolePixel) {
    // off-resonance in the row-padded pixel layout, and its difference to
    // the centre of the 16-pixel tile
    if (i >= a.Rp) return;
    const int rq = (int)i;
    const double v = pixel_dw(dw0, rq, a.nx, a.ny, a.nxq);
    a.dwq[pz * a.Rp + rq] = v;
    if (a.ddw) a.ddw[pz * a.Rp + rq] = (float)(v - pixel_dw(dw0, (rq & ~15) + 8, a.nx, a.ny, a.nxq));
    return;
  }
  if (role == kRoleSq) {
    // sq[row][col] = S_col(r) in the adjoint's partial-sum layout, zero on
    // padding rows and columns
    if (i >= (int64_t)a.Rp * a.NCP) return;
    const int row = (int)(i / a.NCP), col = (int)(i % a.NCP);
    const int yy = row / a.nxq, xx = row - yy * a.nxq;
    float2 v = make_float2(0.f, 0.f);
    if (col < a.C && xx < a.nx && yy < a.ny) v = a.smaps[(pz * a.C + col) * a.R + (int64_t)yy * a.nx + xx];
    a.sq[pz * a.Rp * a.NCP + i] = v;
    return;
  }
  if (role == kRoleKap) {
    // general basis, samples: (k_l(t)/2pi, t) and the FP32 difference to the
    // centre of the 16-sample tile
    if (i >= a.Tp * a.NT) return;
    const int64_t t = i / a.NT;
    const int j = (int)(i - t * a.NT);
    auto val = [&](int64_t s) -> double {
      s = min(s, a.T - 1);
      return j < a.L ? coef[s * a.L + j] * kInv2Pi : j == a.L ? time[s] : 0.0;
    };
    const double v = val(t);
    a.kap[(pz * a.Tp + t) * a.NT + j] = v;
    if (a.dkap) put_diff(a.dkap + pz * a.Tp * nte, t, j, a.NT, (float)(v - val((t & ~int64_t(15)) + 8)));
    return;
  }
  if (role == kRoleBet) {
    // general basis, pixels: (b_l(r), dw0/2pi), and the difference as above
    if (i >= (int64_t)a.Rp * a.NT) return;
    const int r = (int)(i / a.NT), j = (int)(i - (int64_t)r * a.NT);
    const double *basis = a.basis ? a.basis + pz * a.L * a.R : nullptr;
    auto val = [&](int s) -> double {
      s = min(s, a.R - 1);
      return j < a.L ? basis[(int64_t)j * a.R + s] : j == a.L && dw0 ? dw0[s] * kInv2Pi : 0.0;
    };
    const double v = val(r);
    a.bet[(pz * a.Rp + r) * a.NT + j] = v;
    if (a.dbet) put_diff(a.dbet + pz * a.Rp * nte, r, j, a.NT, (float)(v - val((r & ~15) + 8)));
    return;
  }
  // magnitude bounds of the scaled forms, per workgroup: |Re| + |Im| of the coil
  // maps (third section) and of an image operand, the larger component of a
  // data operand (first section)
  const bool maps = role == kRoleMaps;
  const float2 *v = maps ? a.smaps + pz * a.C * a.R : a.operand + pz * a.nop;
  const int64_t n = maps ? (int64_t)a.C * a.R : a.nop;
  const bool l1 = maps || a.op_l1;
  float m = 0.f;
  const int nblk = (int)(a.end[role] - a.end[role - 1]);
  for (int64_t k = (int64_t)blk * 256 + tid; k < n; k += (int64_t)nblk * 256) {
    m = fmaxf(m, magnitude(v[k], l1));
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((tid & 63) == 0) wm[tid >> 6] = m;
  __syncthreads();
  const int slot = (int)blk + tid * nblk;
  if (slot < kAmaxBlocks)
    a.amax[((maps ? 2 * (int64_t)gridDim.y : 0) + pz) * kAmaxBlocks + slot] = fmaxf(fmaxf(wm[0], wm[1]),
                                                                                    fmaxf(wm[2], wm[3]));
}

int enc_prepare(const EncPlan &p, const expenc_op *op, const EncBuffers &b, hipStream_t s, int need,
                const float2 *operand) {
  const bool split = p.prec != EXPENC_FP32;
  const bool fwd = (need & kNeedForward) != 0, adj = (need & kNeedAdjoint) != 0;
  PrepArgs a{};
  a.coef = op->coef;
  a.time = op->time;
  a.basis = op->basis;
  a.dw0 = op->dw0;
  a.z0s = p.z0s;
  a.smaps = reinterpret_cast<const float2 *>(op->smaps);
  a.operand = operand;
  a.T = p.T;
  a.Tp = p.Tp;
  a.R = p.R;
  a.Rp = p.Rp;
  a.L = p.L;
  a.NT = p.NT;
  a.nx = p.nx;
  a.ny = p.ny;
  a.nxq = p.nxq;
  a.C = p.C;
  a.NCP = p.NCP;
  a.dx = p.dx;
  a.dy = p.dy;
  a.z0 = p.z0;
  a.nop = fwd ? (int64_t)p.B * p.R : p.T * p.NC;
  a.op_l1 = fwd;
  int64_t n[kRoles] = {};
  if (p.sh) {
    a.pmono = b.pmono;
    a.dwq = b.dwq;
    if (b.pmono) n[kRolePoly] = ceil_div(p.Tp, 256);
    n[kRolePixel] = ceil_div(p.Rp, 256);
    if (split && fwd) a.ddw = b.ddw;
    if (split && adj) {
      if (!b.anc) return fail(EXPENC_EINVAL, "anchor table of a split plan is not carved");
      a.dpa = b.dpa;
      a.anc = b.anc;
      n[kRoleIncr] = ceil_div(p.Tp * 2, 256);
      n[kRoleAnchor] = p.Rp / 256 * ceil_div(p.Tp / 32, kAncTiles);
    }
  } else {
    a.kap = b.kap;
    a.bet = b.bet;
    if (split && fwd) a.dbet = b.dbet;
    if (split && adj) a.dkap = b.dkap;
    n[kRoleKap] = ceil_div(p.Tp * p.NT, 256);
    n[kRoleBet] = ceil_div((int64_t)p.Rp * p.NT, 256);
  }
  if (p.comb && adj) {
    if (!b.sq) return fail(EXPENC_EINVAL, "coil table of a single-image split plan is not carved");
    a.sq = b.sq;
    n[kRoleSq] = ceil_div((int64_t)p.Rp * p.NCP, 256);
  }
  // (the coil maps' bound: also for a bf16 solver's FP32 plan)
  if (b.amax && fwd) {
    a.amax = b.amax;
    n[kRoleMaps] = amax_blocks((int64_t)p.C * p.R);
  }
  if (p.scaled && operand) {
    if (!b.scl || !b.amax || !b.wmax) return fail(EXPENC_EINVAL, "scale buffers of a scaled plan are not carved");
    a.amax = b.amax;
    n[kRoleOperand] = amax_blocks(a.nop);
  } else if (operand) {
    a.NC = p.NC;
    a.rec = reinterpret_cast<u32x4 *>(fwd ? b.zs : b.ys);
    a.rec_image = fwd;
    a.rec_perm = adj || !p.sh;
    a.rec_chunk = fwd ? p.fwd_chunk : p.adj_chunk;
    n[kRoleRecords] = ceil_div((fwd ? p.Rp : p.Tp) * (p.NCP / 4), 256);
  }
  int64_t tot = 0;
  for (int r = 0; r < kRoles; ++r) {
    tot += n[r];
    a.end[r] = (unsigned)tot;
  }
  if (tot > INT32_MAX) return fail(EXPENC_EUNSUPPORTED, "field tables need more than 2^31 workgroups");
  k_prepare<<<dim3((unsigned)tot, (unsigned)p.P), 256, 0, s>>>(a);
  EX_LAUNCHED("field setup");
  return EXPENC_OK;
}

}  // namespace expenc
