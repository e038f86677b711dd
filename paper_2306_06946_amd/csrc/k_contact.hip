// Contact side of the time step: selection of the contacts at the free motion
// (stand-in for collision detection, Sec. "Contact generation"), frames and
// gaps (Eq. 7, 10, 26), the fast compliance update W = C W_H C^T (Eq. 28),
// projected Gauss-Seidel (Eq. 18-19, Algorithm 1), and the proximity update
// p_k = p_free + h^2 W_H C_k^T lambda_k (Eq. 31).
#include <hip/hip_cooperative_groups.h>

#include <algorithm>
#include <mutex>

#include "scene.hpp"

namespace icr {

namespace {

__device__ inline unsigned long long sortable(double x) {
  unsigned long long b = (unsigned long long)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ double signed_distance(const icr_obstacle &o, double t, const double p[3], double nrm[3]) {
#pragma clang fp contract(off)
  double c[3] = {o.c0[0] + o.vel[0] * t, o.c0[1] + o.vel[1] * t, o.c0[2] + o.vel[2] * t};
  double r0 = p[0] - c[0], r1 = p[1] - c[1], r2 = p[2] - c[2];
  if (o.kind == 1) {
    double dist = sqrt(r0 * r0 + r1 * r1 + r2 * r2);
    nrm[0] = r0 / dist;
    nrm[1] = r1 / dist;
    nrm[2] = r2 / dist;
    return dist - o.radius;
  }
  nrm[0] = o.normal[0];
  nrm[1] = o.normal[1];
  nrm[2] = o.normal[2];
  return r0 * o.normal[0] + r1 * o.normal[1] + r2 * o.normal[2];
}

// Exclusive prefix sum of one int per thread over a 1024-thread block.
__device__ int block_excl_scan_1024(int v, int *wsum) {
  const int ln = threadIdx.x & 63, wv = threadIdx.x >> 6;
  int x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(x, o, 64);
    if (ln >= o) x += t;
  }
  if (ln == 63) wsum[wv] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int w = 0; w < 16; ++w) {
      const int t = wsum[w];
      wsum[w] = acc;
      acc += t;
    }
  }
  __syncthreads();
  const int r = wsum[wv] + x - v;
  __syncthreads();
  return r;
}

// Keep the K candidates with smallest (distance, node id) at q_free, in
// ascending node id; gather mu, p_free = H q_free, p_start = H q, warm start.
// The candidate list is ascending by node id (sorted when it is set).  The
// K-th smallest distance key T is found by an MSB-first radix select (8 bits
// per pass, 256-bin histograms in LDS); the contacts are the candidates with
// key < T and the lowest-id ones with key == T, placed by an exclusive scan
// of the selection flags in list order.  Thread t holds list entries
// 4t .. 4t + 3.
constexpr int SEL_PER = 4;   // 4096 candidates at most
__global__ __launch_bounds__(1024) void k_select(int ncand, const int *__restrict__ cand,
                                                 const double *__restrict__ qf, const double *__restrict__ q,
                                                 const StepCtx *__restrict__ ctx, int K,
                                                 const double *__restrict__ mu_node,
                                                 const double *__restrict__ node_force, int *__restrict__ nodes_c,
                                                 double *__restrict__ mu_c, double *__restrict__ pfree,
                                                 double *__restrict__ pstart, double *__restrict__ finit) {
  __shared__ unsigned long long key[1024 * SEL_PER];
  __shared__ int hist[256];
  __shared__ int wsum[16];
  __shared__ unsigned long long s_prefix;
  __shared__ int s_rank;
  const int tid = threadIdx.x, ln = tid & 63, wv = tid >> 6;
  const icr_obstacle obs = ctx->obs;
  const double t1 = ctx->t0 + ctx->h;
#pragma unroll
  for (int e = 0; e < SEL_PER; ++e) {
    const int i = SEL_PER * tid + e;
    unsigned long long kv = ~0ull;
    if (i < ncand) {
      const int v = cand[i];
      double p[3] = {qf[3 * v], qf[3 * v + 1], qf[3 * v + 2]}, nrm[3];
      kv = sortable(signed_distance(obs, t1, p, nrm));
    }
    key[i] = kv;
  }
  if (tid == 0) {
    s_prefix = 0ull;
    s_rank = K;   // rank (1-based) of the sought key among those matching the prefix
  }
  unsigned long long mask = 0ull;
  for (int shift = 56; shift >= 0; shift -= 8) {
    for (int b = tid; b < 256; b += 1024) hist[b] = 0;
    __syncthreads();
    const unsigned long long prefix = s_prefix;
#pragma unroll
    for (int e = 0; e < SEL_PER; ++e) {
      const int i = SEL_PER * tid + e;
      if (i < ncand && (key[i] & mask) == prefix) atomicAdd(&hist[(int)((key[i] >> shift) & 255ull)], 1);
    }
    __syncthreads();
    if (wv == 0) {
      const int c0 = hist[4 * ln], c1 = hist[4 * ln + 1], c2 = hist[4 * ln + 2], c3 = hist[4 * ln + 3];
      const int tot = c0 + c1 + c2 + c3;
      int incl = tot;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (ln >= o) incl += t;
      }
      const int rank = s_rank;
      int run = incl - tot;
      const int c[4] = {c0, c1, c2, c3};
      for (int qd = 0; qd < 4; ++qd) {
        if (run < rank && rank <= run + c[qd]) {   // exactly one bin of the wave
          s_prefix = prefix | ((unsigned long long)(4 * ln + qd) << shift);
          s_rank = rank - run;
        }
        run += c[qd];
      }
    }
    __syncthreads();
    mask |= 0xffull << shift;
  }
  const unsigned long long T = s_prefix;
  const int need = s_rank;   // candidates with key == T to keep, lowest ids first
  int tf[SEL_PER], tsum = 0;
#pragma unroll
  for (int e = 0; e < SEL_PER; ++e) {
    const int i = SEL_PER * tid + e;
    tf[e] = (i < ncand && key[i] == T) ? 1 : 0;
    tsum += tf[e];
  }
  int tr = block_excl_scan_1024(tsum, wsum);
  int sf[SEL_PER], ssum = 0;
#pragma unroll
  for (int e = 0; e < SEL_PER; ++e) {
    const int i = SEL_PER * tid + e;
    sf[e] = (i < ncand && (key[i] < T || (tf[e] && tr < need))) ? 1 : 0;
    tr += tf[e];
    ssum += sf[e];
  }
  int c = block_excl_scan_1024(ssum, wsum);
#pragma unroll
  for (int e = 0; e < SEL_PER; ++e) {
    if (!sf[e]) continue;
    const int v = cand[SEL_PER * tid + e];
    nodes_c[c] = v;
    mu_c[c] = mu_node[v];
    for (int a = 0; a < 3; ++a) {
      pfree[3 * c + a] = qf[3 * v + a];
      pstart[3 * c + a] = q[3 * v + a];
      finit[3 * c + a] = node_force[3 * v + a];
    }
    ++c;
  }
}

// Frame (rows n, t1, t2: normal and axis-rule tangents) and gap delta of a
// contact at proximity pc: normal gap = signed distance at t1, tangential gap
// = relative tangential displacement over the step.
__device__ inline void contact_frame(const icr_obstacle &obs, double t0, double t1, const double pc[3],
                                     const double ps[3], double F[3][3], double delta[3]) {
  double n[3];
  double phi = signed_distance(obs, t1, pc, n);
  int ax = 0;
  double am = fabs(n[0]);
  if (fabs(n[1]) < am) {
    ax = 1;
    am = fabs(n[1]);
  }
  if (fabs(n[2]) < am) ax = 2;
  double en = n[ax];
  double ta[3] = {-en * n[0], -en * n[1], -en * n[2]};
  ta[ax] += 1.0;
  double tn = sqrt(ta[0] * ta[0] + ta[1] * ta[1] + ta[2] * ta[2]);
  ta[0] /= tn;
  ta[1] /= tn;
  ta[2] /= tn;
  double tb[3] = {n[1] * ta[2] - n[2] * ta[1], n[2] * ta[0] - n[0] * ta[2], n[0] * ta[1] - n[1] * ta[0]};
  double rel[3];
  for (int a = 0; a < 3; ++a) {
    double uo = (obs.c0[a] + obs.vel[a] * t1) - (obs.c0[a] + obs.vel[a] * t0);
    rel[a] = pc[a] - ps[a] - uo;
  }
  for (int a = 0; a < 3; ++a) {
    F[0][a] = n[a];
    F[1][a] = ta[a];
    F[2][a] = tb[a];
  }
  delta[0] = phi;
  delta[1] = ta[0] * rel[0] + ta[1] * rel[1] + ta[2] * rel[2];
  delta[2] = tb[0] * rel[0] + tb[1] * rel[1] + tb[2] * rel[2];
}

// Frame and gap of a pair contact between two bodies: the given normal n of
// the second body's surface (fixed over the step), tangents by the axis
// rule, normal gap n . p of the relative position p = x_1 - x_2, tangential
// gap = relative tangential displacement over the step.
__device__ inline void pair_frame(const double n[3], const double pc[3], const double ps[3], double F[3][3],
                                  double delta[3]) {
  int ax = 0;
  double am = fabs(n[0]);
  if (fabs(n[1]) < am) {
    ax = 1;
    am = fabs(n[1]);
  }
  if (fabs(n[2]) < am) ax = 2;
  double en = n[ax];
  double ta[3] = {-en * n[0], -en * n[1], -en * n[2]};
  ta[ax] += 1.0;
  double tn = sqrt(ta[0] * ta[0] + ta[1] * ta[1] + ta[2] * ta[2]);
  ta[0] /= tn;
  ta[1] /= tn;
  ta[2] /= tn;
  double tb[3] = {n[1] * ta[2] - n[2] * ta[1], n[2] * ta[0] - n[0] * ta[2], n[0] * ta[1] - n[1] * ta[0]};
  double rel[3] = {pc[0] - ps[0], pc[1] - ps[1], pc[2] - ps[2]};
  for (int a = 0; a < 3; ++a) {
    F[0][a] = n[a];
    F[1][a] = ta[a];
    F[2][a] = tb[a];
  }
  delta[0] = n[0] * pc[0] + n[1] * pc[1] + n[2] * pc[2];
  delta[1] = ta[0] * rel[0] + ta[1] * rel[1] + ta[2] * rel[2];
  delta[2] = tb[0] * rel[0] + tb[1] * rel[1] + tb[2] * rel[2];
}

// Frames C_k and gaps at p_{k-1}; d_k = delta - C_k (p - p_free); warm start
// lambda = C_k f with f the previous world-frame force.  The first npair
// contacts are pairs with normals pn.
__device__ __forceinline__ void directions_contact(int c, const StepCtx *__restrict__ ctx, const double *__restrict__ p,
                                                   const double *__restrict__ pfree,
                                                   const double *__restrict__ pstart,
                                                   const double *__restrict__ fprev, double *__restrict__ C,
                                                   double *__restrict__ dk, double *__restrict__ lam, int npair,
                                                   const double *__restrict__ pn) {
  const icr_obstacle obs = ctx->obs;
  const double t0 = ctx->t0, t1 = ctx->t0 + ctx->h;
  double pc[3] = {p[3 * c], p[3 * c + 1], p[3 * c + 2]};
  double ps[3] = {pstart[3 * c], pstart[3 * c + 1], pstart[3 * c + 2]};
  double F[3][3], delta[3];
  if (c < npair) {
    const double n[3] = {pn[3 * c], pn[3 * c + 1], pn[3 * c + 2]};
    pair_frame(n, pc, ps, F, delta);
  } else {
    contact_frame(obs, t0, t1, pc, ps, F, delta);
  }
  double dp[3] = {pc[0] - pfree[3 * c], pc[1] - pfree[3 * c + 1], pc[2] - pfree[3 * c + 2]};
  for (int r = 0; r < 3; ++r) {
    for (int a = 0; a < 3; ++a) C[9 * c + 3 * r + a] = F[r][a];
    dk[3 * c + r] = delta[r] - (F[r][0] * dp[0] + F[r][1] * dp[1] + F[r][2] * dp[2]);
    lam[3 * c + r] = F[r][0] * fprev[3 * c] + F[r][1] * fprev[3 * c + 1] + F[r][2] * fprev[3 * c + 2];
  }
}
__global__ void k_directions(int nc, const StepCtx *__restrict__ ctx, const double *__restrict__ p,
                             const double *__restrict__ pfree, const double *__restrict__ pstart,
                             const double *__restrict__ fprev, double *__restrict__ C, double *__restrict__ dk,
                             double *__restrict__ lam, int npair, const double *__restrict__ pn) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < nc) directions_contact(c, ctx, p, pfree, pstart, fprev, C, dk, lam, npair, pn);
}

// W_ab = C_a (W_H)_ab C_b^T.  Block (a, b) with a < b is computed as the
// transpose of block (b, a) from the same inputs (W_H is exactly symmetric),
// so W is exactly symmetric.
template <class TW>
__device__ __forceinline__ void update_W_block(int nc, const TW *__restrict__ WH, const double *__restrict__ C,
                                               TW *__restrict__ W, long blk) {
  const int a = (int)(blk / nc), b = (int)(blk % nc);
  const long m = 3L * nc;
  const bool lower = a >= b;
  double M[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double v = (double)WH[(3L * a + i) * m + 3L * b + j];
      if (lower)
        M[i][j] = v;
      else
        M[j][i] = v;
    }
  const double *X = C + 9L * (lower ? a : b);
  const double *Y = C + 9L * (lower ? b : a);
  double T[3][3];   // M Y^T
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) T[i][j] = M[i][0] * Y[3 * j] + M[i][1] * Y[3 * j + 1] + M[i][2] * Y[3 * j + 2];
  double R[3][3];   // X T
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) R[i][j] = X[3 * i] * T[0][j] + X[3 * i + 1] * T[1][j] + X[3 * i + 2] * T[2][j];
  // diagonal blocks: mirror the lower entries so the block is exactly symmetric
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double v;
      if (a == b)
        v = (i >= j) ? R[i][j] : R[j][i];
      else
        v = lower ? R[i][j] : R[j][i];
      W[(3L * a + i) * m + 3L * b + j] = (TW)v;
    }
}

template <class TW>
__global__ void k_update_W(int nc, const TW *__restrict__ WH, const double *__restrict__ C, TW *__restrict__ W) {
  const long blk = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (blk < (long)nc * nc) update_W_block(nc, WH, C, W, blk);
}

// ---- local solver (Signorini + Coulomb cone) --------------------------------

struct Local {
  double l[3];
  int st;
};

__device__ Local local_solve(const double w[3][3], const double d[3], double mu, int j_inner) {
  Local out;
  if (d[0] >= 0.0) {
    out.l[0] = out.l[1] = out.l[2] = 0.0;
    out.st = ICR_SEPARATE;
    return out;
  }
  // stick trial: 3x3 Cholesky solve
  double l00 = sqrt(w[0][0]);
  double l10 = w[1][0] / l00, l20 = w[2][0] / l00;
  double l11 = sqrt(w[1][1] - l10 * l10);
  double l21 = (w[2][1] - l20 * l10) / l11;
  double l22 = sqrt(w[2][2] - l20 * l20 - l21 * l21);
  double y0 = d[0] / l00;
  double y1 = (d[1] - l10 * y0) / l11;
  double y2 = (d[2] - l20 * y0 - l21 * y1) / l22;
  double x2 = y2 / l22;
  double x1 = (y1 - l21 * x2) / l11;
  double x0 = (y0 - l10 * x1 - l20 * x2) / l00;
  double ln = -x0, lt1 = -x1, lt2 = -x2;
  if (ln > 0.0 && lt1 * lt1 + lt2 * lt2 <= (mu * ln) * (mu * ln)) {
    out.l[0] = ln;
    out.l[1] = lt1;
    out.l[2] = lt2;
    out.st = ICR_STICK;
    return out;
  }
  double u0, u1;
  double nt = sqrt(lt1 * lt1 + lt2 * lt2);
  if (nt > 0.0) {
    u0 = lt1 / nt;
    u1 = lt2 / nt;
  } else {
    double ndt = sqrt(d[1] * d[1] + d[2] * d[2]);
    if (ndt > 0.0) {
      u0 = -d[1] / ndt;
      u1 = -d[2] / ndt;
    } else {
      u0 = 1.0;
      u1 = 0.0;
    }
  }
  const double kap = 0.5 * (w[1][1] + w[2][2]);
  for (int it = 0; it < j_inner; ++it) {
    double den = w[0][0] + mu * (w[0][1] * u0 + w[0][2] * u1);
    if (den <= 0.0) den = w[0][0];
    double lam_n = -d[0] / den;
    double a1 = mu * lam_n * u0, a2 = mu * lam_n * u1;
    double r1 = d[1] + w[1][0] * lam_n + (w[1][1] - kap) * a1 + w[1][2] * a2;
    double r2 = d[2] + w[2][0] * lam_n + w[2][1] * a1 + (w[2][2] - kap) * a2;
    double nr = sqrt(r1 * r1 + r2 * r2);
    if (nr > 0.0) {
      u0 = -r1 / nr;
      u1 = -r2 / nr;
    }
  }
  double den = w[0][0] + mu * (w[0][1] * u0 + w[0][2] * u1);
  if (den <= 0.0) den = w[0][0];
  double lam_n = -d[0] / den;
  out.l[0] = lam_n;
  out.l[1] = mu * lam_n * u0;
  out.l[2] = mu * lam_n * u1;
  out.st = ICR_SLIP;
  return out;
}

// 1/x and 1/sqrt(x) from the hardware estimates refined by two Newton steps
// (full double precision for the well-scaled positive values used here).
__device__ inline double frcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ inline double frsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
// One Newton step only: relative error about the square of the estimate's
// (used inside the slip fixed point, whose iterates are renormalised anyway).
__device__ inline double frsqrt1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

// Per-contact record of the Gauss-Seidel chains, computed once per active set
// from the symmetric 3x3 block w of h^2 W_aa and mu.  Everything the slip
// passes use is divided by w00, so that a pass needs no product with it:
//   i..    the entries of -w^-1 (the stick trial is -w^-1 d)
//   it00   1 / w00, negated when w00 <= mu |(w01, w02)| (with margin): only
//          with the margin is den(u) > 0 on the whole unit circle, and only
//          then does the slip pass need no fallback
//   wh0/1  w01 / w00, w02 / w00
//   a2/b2  2 mu wh0, 2 mu wh1
//   m11    2 mu (w11 - kappa) / w00 = -2 mu (w22 - kappa) / w00, kappa = (w11 + w22) / 2
//   m12    2 mu w12 / w00
// FAST (a record built inside a Gauss-Seidel visit, on its dependent chain):
// refined reciprocals and the margin test compared squared.
constexpr int PGS_RW = kPgsRecWidth;   // rows of a stored record: these 14, then up to 6 of the caller's
struct PgsRec {
  double i00, i01, i02, i11, i12, i22, mu, it00, wh0, wh1, a2, b2, m11, m12;
};
constexpr int PGS_RC = 14;
static_assert(sizeof(PgsRec) == PGS_RC * sizeof(double) && PGS_RW == PGS_RC + 6, "record rows");
template <bool FAST = false>
__device__ __forceinline__ PgsRec make_record(const double w[3][3], double mu) {
  PgsRec r;
  const double w00 = w[0][0], w01 = w[0][1], w02 = w[0][2], w11 = w[1][1], w12 = w[1][2], w22 = w[2][2];
  const double c00 = w11 * w22 - w12 * w12, c01 = w02 * w12 - w01 * w22, c02 = w01 * w12 - w02 * w11;
  const double c11 = w00 * w22 - w02 * w02, c12 = w01 * w02 - w00 * w12, c22 = w00 * w11 - w01 * w01;
  const double det = w00 * c00 + w01 * c01 + w02 * c02;
  const double idet = FAST ? frcp(det) : 1.0 / det;
  const double i00 = FAST ? frcp(w00) : 1.0 / w00;
  r.i00 = -(c00 * idet);
  r.i01 = -(c01 * idet);
  r.i02 = -(c02 * idet);
  r.i11 = -(c11 * idet);
  r.i12 = -(c12 * idet);
  r.i22 = -(c22 * idet);
  r.mu = mu;
  bool safe;
  if (FAST) {
    const double mm = 1.000001 * mu;   // w00 > mm |(w01, w02)| squared, w00 > 0
    safe = w00 > 0.0 && w00 * w00 > (mm * mm) * (w01 * w01 + w02 * w02);
  } else {
    safe = w00 > 1.000001 * mu * sqrt(w01 * w01 + w02 * w02);
  }
  r.it00 = safe ? i00 : -fabs(i00);
  r.wh0 = w01 * i00;
  r.wh1 = w02 * i00;
  const double m2 = 2.0 * mu;
  r.a2 = m2 * r.wh0;
  r.b2 = m2 * r.wh1;
  r.m11 = m2 * (0.5 * (w11 - w22)) * i00;
  r.m12 = m2 * w12 * i00;
  return r;
}

// Guarded slip pass (rare: the record's den > 0 guarantee fails, |v| = 0
// occurred, or the unnormalised iterate left the safe range): den <= 0
// replaced by w_nn as in the direct form, |v| = 0 keeps the direction;
// restarts from the initial direction and normalises every pass.
struct SlipIn {
  double wh0, wh1, a2, b2, m11, m12;    // record entries
  double d0, d1, d2, lt1, lt2, nt2;     // gap, stick trial
};
__device__ __forceinline__ double2 guarded_slip(const SlipIn a, int j_inner) {
  double u0, u1;
  if (a.nt2 > 0.0) {
    const double inv = frsqrt(a.nt2);
    u0 = a.lt1 * inv;
    u1 = a.lt2 * inv;
  } else {
    const double nd2 = a.d1 * a.d1 + a.d2 * a.d2;
    if (nd2 > 0.0) {
      const double inv = frsqrt(nd2);
      u0 = -a.d1 * inv;
      u1 = -a.d2 * inv;
    } else {
      u0 = 1.0;
      u1 = 0.0;
    }
  }
  const double al = 0.5 * a.a2, be = 0.5 * a.b2, m11 = 0.5 * a.m11, m12 = 0.5 * a.m12;
  for (int it = 0; it < j_inner; ++it) {
    // -r(u) up to a positive factor: d_n e(u) - den(u) d_t over w00
    double den = fma(al, u0, fma(be, u1, 1.0));
    if (!(den > 0.0)) den = 1.0;
    const double e1 = fma(m11, u0, fma(m12, u1, a.wh0)), e2 = fma(m12, u0, fma(-m11, u1, a.wh1));
    const double v0 = fma(a.d0, e1, -den * a.d1), v1 = fma(a.d0, e2, -den * a.d2);
    const double s2 = v0 * v0 + v1 * v1;
    if (s2 > 0.0) {
      const double inv = frsqrt(s2);
      u0 = v0 * inv;
      u1 = v1 * inv;
    }
  }
  return make_double2(u0, u1);
}

// The local solve of one Gauss-Seidel visit, run by a whole wave: every lane
// works on its own record and gap, and the branches follow the lane li whose
// contact is visited, so control flow is uniform and the other lanes' values
// are unused.  Same branches and fixed point as local_solve, from the record:
// stick trial by the precomputed inverse, refined reciprocals instead of
// divisions, and the slip pass on the direction alone.  With den(u) =
// 1 + al u0 + be u1 > 0 (over w00; al = a2 / 2, be = b2 / 2) the tangential
// residual r = d_t + lam_n(u) e(u), lam_n = -d_n / (w00 den(u)),
// e(u) = w_tn + mu (W_tt - kappa I) u, gives the direction
//   -r / |r| = v / |v|,   v(u) = n + N u,
//   n = d_n w_tn / w00 - d_t,   N = d_n mu (W_tt - kappa I) / w00 - d_t (al, be).
// A pass is u <- v(u) / |v(u)|.  The iterate is kept unnormalised: with
// u = v / r, r = |v|, the next one is taken as v' = n (2 r) + (2 N) v, which
// has the same direction (12 instructions and no reciprocal; the normalised
// form took 13, and 11 more for the start direction: the stick trial's
// tangential part is a start as it is).  The magnitude is multiplied by
// 2 |n + N u| in each pass; when it has left 1e-125 .. 1e125 after the last
// one, the guarded pass runs instead.  What bounds a visit is one wave's issue
// rate: whatever its dependences, an instruction of 4 bytes takes 5 cycles
// and one of 8 bytes 6, an rsq or rcp 17, a taken branch 22, a scalar
// instruction that reads a comparison's mask at once 16 more (measured, one
// wave on its SIMD).  So every form here is chosen for its instruction count
// and size; a pass takes 68 cycles.
// J = 8: the default pass count, straight-line; J = 0: j_inner passes in a
// loop, normalised (their number is not bounded).
// `bit` selects the visited lane in the masks.
__device__ __forceinline__ bool lane_in(unsigned long long mask, unsigned long long bit) { return (mask & bit) != 0; }
struct Trial {
  double ln, lt1, lt2, nt2;
  double p, q;                // d_n m11, d_n m12 of the slip passes
  unsigned long long stick;   // lanes whose trial lies inside the cone
};
__device__ __forceinline__ Trial stick_trial(const PgsRec &rc, double d0, double d1, double d2) {
  Trial t;
  t.ln = fma(rc.i02, d2, fma(rc.i01, d1, rc.i00 * d0));
  t.lt1 = fma(rc.i12, d2, fma(rc.i11, d1, rc.i01 * d0));
  t.lt2 = fma(rc.i22, d2, fma(rc.i12, d1, rc.i02 * d0));
  t.nt2 = fma(t.lt1, t.lt1, t.lt2 * t.lt2);
  const double ml = rc.mu * t.ln;
  const bool in = t.nt2 <= ml * ml, pos = t.ln > 0.0;
  t.p = d0 * rc.m11;
  t.q = d0 * rc.m12;
  // A scalar instruction waits some 16 cycles for a comparison's mask: the
  // two products, which only the slip passes use, are issued meanwhile.
  asm("" : "+v"(t.p), "+v"(t.q));
  t.stick = __ballot(in) & __ballot(pos);
  return t;
}
template <int J>
__device__ __forceinline__ void slip_solve(const PgsRec &rc, const Trial &tr, double d0, double d1, double d2,
                                           int j_inner, unsigned long long bit, unsigned long long safe,
                                           double (&l)[3]) {
  const double t = -d0 * fabs(rc.it00);
  const double n0 = fma(d0, rc.wh0, -d1), n1 = fma(d0, rc.wh1, -d2);
  const double p = tr.p, q = tr.q;
  const double M00 = fma(-d1, rc.a2, p), M01 = fma(-d1, rc.b2, q);   // 2 N
  const double M10 = fma(-d2, rc.a2, q), M11 = fma(-d2, rc.b2, -p);
  double v0 = tr.lt1, v1 = tr.lt2, s = tr.nt2;
  if constexpr (J == 8) {
#pragma unroll
    for (int it = 0; it < 8; ++it) {
      // R = 2 |v|: the estimate s y of |v| refined by one Newton step; two
      // products cover the wait state that the estimate's first use needs
      const double y = __builtin_amdgcn_rsq(s);
      __builtin_amdgcn_sched_barrier(0);
      const double a0 = M01 * v1, a1 = M11 * v1;
      __builtin_amdgcn_sched_barrier(0);
      const double r0 = s * y;
      const double R = r0 * fma(-r0, y, 3.0);
      const double x0 = fma(n0, R, fma(M00, v0, a0));
      const double x1 = fma(n1, R, fma(M10, v0, a1));
      v0 = x0;
      v1 = x1;
      s = fma(v0, v0, v1 * v1);
    }
  } else {
    const double inv0 = frsqrt(tr.nt2);
    v0 *= inv0;
    v1 *= inv0;
    for (int it = 0; it < j_inner; ++it) {
      const double x0 = fma(0.5 * M00, v0, fma(0.5 * M01, v1, n0));
      const double x1 = fma(0.5 * M10, v0, fma(0.5 * M11, v1, n1));
      const double inv = frsqrt1(fma(x0, x0, x1 * x1));
      v0 = x0 * inv;
      v1 = x1 * inv;
    }
    s = fma(v0, v0, v1 * v1);
  }
  // r = |v| and 1 / D by one third-order step each; lam_n = t / den(u),
  // lam_t = mu lam_n v / r with den(u) = D / (2 r)
  const double y = __builtin_amdgcn_rsq(s);
  const double r0 = s * y;
  const double e = fma(-r0, y, 1.0);
  const double r = fma(r0, fma(e, 0.375, 0.5) * e, r0);
  const double rr = r + r;
  const double D = fma(rc.a2, v0, fma(rc.b2, v1, rr));
  const double z = __builtin_amdgcn_rcp(D);
  const double c = fma(-D, z, 1.0);
  const double g = t * fma(z, fma(c, c, c), z);
  const double k = (rc.mu + rc.mu) * g;
  l[0] = g * rr;
  l[1] = k * v0;
  l[2] = k * v1;
  // a zero, a NaN or a magnitude near the ends of the range fails this
  if (__builtin_expect(!lane_in(safe & __ballot(s > 1e-250) & __ballot(s < 1e250), bit), 0)) {
    const SlipIn a{rc.wh0, rc.wh1, rc.a2, rc.b2, rc.m11, rc.m12, d0, d1, d2, tr.lt1, tr.lt2, tr.nt2};
    const double2 u = guarded_slip(a, j_inner);
    double den = 0.5 * fma(rc.a2, u.x, fma(rc.b2, u.y, 2.0));
    if (den <= 0.0) den = 1.0;
    const double lam_n = t * frcp(den);
    const double mln = rc.mu * lam_n;
    l[0] = lam_n;
    l[1] = mln * u.x;
    l[2] = mln * u.y;
  }
}
// One contact's solve where every lane holds the same values.
template <int J>
__device__ __forceinline__ Local local_solve_rec(const PgsRec &rc, const double d[3], int j_inner) {
  Local out;
  out.l[0] = out.l[1] = out.l[2] = 0.0;
  out.st = ICR_SEPARATE;
  if (lane_in(__ballot(d[0] >= 0.0), 1ull)) return out;
  const Trial t = stick_trial(rc, d[0], d[1], d[2]);
  if (lane_in(t.stick, 1ull)) {
    out.l[0] = t.ln;
    out.l[1] = t.lt1;
    out.l[2] = t.lt2;
    out.st = ICR_STICK;
  } else {
    slip_solve<J>(rc, t, d[0], d[1], d[2], j_inner, 1ull, __ballot(rc.it00 > 0.0), out.l);
    out.st = ICR_SLIP;
  }
  return out;
}

// Deterministic block reduction of one double (1024 threads).
__device__ double block_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += red[i];
  return s;   // valid in thread 0
}

// Deterministic block reductions over the active-set kernel's threads (valid
// in thread 0): three sums at once, and a minimum.
__device__ void block_sum3(double &a, double &b, double &c, double *red) {
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
    c += __shfl_xor(c, o, 64);
  }
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, nw = (int)(blockDim.x >> 6);
  __syncthreads();
  if (l == 0) {
    red[w] = a;
    red[16 + w] = b;
    red[32 + w] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = b = c = 0.0;
    for (int i = 0; i < nw; ++i) {
      a += red[i];
      b += red[16 + i];
      c += red[32 + i];
    }
  }
}
__device__ double block_min(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, nw = (int)(blockDim.x >> 6);
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  double r = INFINITY;
  if (threadIdx.x == 0)
    for (int i = 0; i < nw; ++i) r = fmin(r, red[i]);
  return r;
}

// g0 = d + h^2 W lambda0, one wave per row (the PGS start state).
// y = x0 + h2 M v for a symmetric m x m row-major M (m = 3 nc) and a vector v
// that is non-zero on few contacts (3-blocks of v): by symmetry
// (M v)_i = sum over contacts k with a non-zero block of M[3k+a][i] v[3k+a],
// so only those rows of M are read, each contiguous in the output index i.
// A skipped term is an exact zero, so only the summation order differs from
// the dense product.  Every block compacts the non-zero contacts (ascending,
// SG_CHUNK at a time) into LDS, then its waves split that list over the same
// 64 outputs and add their partial sums in a fixed order.
// World-frame force of contact c from its frame rows and force components.
__device__ inline double world_force(const double *__restrict__ C, const double *__restrict__ lam, long c, int a) {
  const double *R = C + 9 * c;
  return R[a] * lam[3 * c] + R[3 + a] * lam[3 * c + 1] + R[6 + a] * lam[3 * c + 2];
}

constexpr int SG_NT = 512;
constexpr int SG_NW = SG_NT / 64;
constexpr int SG_CHUNK = 2048;
__device__ inline bool block_nonzero(const double *__restrict__ v, long c) {
  return (v[3 * c] != 0.0) | (v[3 * c + 1] != 0.0) | (v[3 * c + 2] != 0.0);
}
// With C given, the vector is the world-frame force f = C^T lambda of the
// contacts (v is then ignored): every block forms the entries it needs from
// C and lambda, and block 0 also writes f for all contacts to fout.
template <class TM>
__device__ __forceinline__ void sym_gemv_sparse(int nc, const TM *__restrict__ M, const double *__restrict__ x0,
                                                const double *__restrict__ v, double h2, double *__restrict__ y,
                                                const double *__restrict__ C, const double *__restrict__ lam,
                                                double *__restrict__ fout) {
  __shared__ int list[SG_CHUNK];
  __shared__ double fl[3 * SG_CHUNK];   // world forces of the listed contacts (with C)
  __shared__ int wsum[SG_NW];
  __shared__ double part[SG_NW][64];
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const long m = 3L * nc;
  const long i = (long)blockIdx.x * 64 + ln;
  const double *nzv = C ? lam : v;   // same zero blocks: C is a rotation
  if (C && blockIdx.x == 0)
    for (long e = tid; e < m; e += SG_NT) fout[e] = world_force(C, lam, e / 3, (int)(e % 3));
  double s = 0.0;
  for (int c0 = 0; c0 < nc; c0 += SG_CHUNK) {
    const int cn = min(SG_CHUNK, nc - c0);
    const int per = (cn + SG_NT - 1) / SG_NT;   // contiguous contacts per thread
    const int lo = c0 + min(cn, tid * per), hi = c0 + min(cn, (tid + 1) * per);
    int cnt = 0;
    for (int c = lo; c < hi; ++c) cnt += block_nonzero(nzv, c) ? 1 : 0;
    int incl = cnt;   // inclusive scan over the wave, then over the waves
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (ln >= o) incl += t;
    }
    if (ln == 63) wsum[wv] = incl;
    __syncthreads();
    int pos = incl - cnt, total = 0;
    for (int w = 0; w < SG_NW; ++w) {
      pos += (w < wv) ? wsum[w] : 0;
      total += wsum[w];
    }
    for (int c = lo; c < hi; ++c)
      if (block_nonzero(nzv, c)) list[pos++] = c;
    __syncthreads();
    if (C) {
      for (int e = tid; e < 3 * total; e += SG_NT) fl[e] = world_force(C, lam, list[e / 3], e % 3);
      __syncthreads();
    }
    if (i < m) {
#pragma unroll 4
      for (int q = wv; q < total; q += SG_NW) {
        const long r = 3L * list[q];
        const double v0 = C ? fl[3 * q] : v[r], v1 = C ? fl[3 * q + 1] : v[r + 1], v2 = C ? fl[3 * q + 2] : v[r + 2];
        s = fma((double)M[r * m + i], v0, s);
        s = fma((double)M[(r + 1) * m + i], v1, s);
        s = fma((double)M[(r + 2) * m + i], v2, s);
      }
    }
    __syncthreads();   // list and wsum are rewritten by the next chunk
  }
  part[wv][ln] = s;
  __syncthreads();
  if (wv == 0 && i < m) {
    double t = 0.0;
    for (int w = 0; w < SG_NW; ++w) t += part[w][ln];
    y[i] = x0[i] + h2 * t;
  }
}
template <class TM>
__global__ __launch_bounds__(SG_NT) void k_sym_gemv_sparse(int nc, const TM *__restrict__ M,
                                                           const double *__restrict__ x0,
                                                           const double *__restrict__ v, double h2,
                                                           double *__restrict__ y, const double *__restrict__ C,
                                                           const double *__restrict__ lam,
                                                           double *__restrict__ fout) {
  sym_gemv_sparse<TM>(nc, M, x0, v, h2, y, C, lam, fout);
}

// Single-workgroup PGS.  g = d + W~ lambda (all contacts, own term included)
// lives in LDS; for contact a: d_a = g_a - W~_aa lambda_a, local solve, then
// g += W~[:, a] (lambda_new - lambda_old), read from rows of the exactly
// symmetric W.  A contact whose force is zero and whose gap g_n is >= 0 is a
// no-op of Gauss-Seidel (it stays separated and changes nothing), so wave 0
// scans 64 contacts at a time with a ballot and jumps to the first contact
// that can change; the iterates are those of the sequential sweep.
constexpr int PGS_MAX_NC = 4096;
// dynamic LDS of k_pgs_single: g[3 nc] doubles, then nz[nc] bytes
__host__ __device__ inline size_t pgs_single_lds(int nc) { return (size_t)nc * (3 * sizeof(double) + 1); }
template <class TW>
__global__ __launch_bounds__(1024) void k_pgs_single(int nc, const TW *__restrict__ W,
                                                     const double *__restrict__ d, const double *__restrict__ g0,
                                                     const double *__restrict__ mu, double h2,
                                                     double *__restrict__ lam, int8_t *__restrict__ status,
                                                     int max_sweeps, double tol, int j_inner,
                                                     int *__restrict__ sweeps_out, double *__restrict__ eps_out,
                                                     const int *__restrict__ ctl) {
  extern __shared__ double lds_g[];
  double *g = lds_g;
  unsigned char *nz = reinterpret_cast<unsigned char *>(lds_g + 3 * nc);
  __shared__ double bc[3];
  __shared__ double red[16];
  __shared__ int ctl_s;
  __shared__ int stop;
  // resume mode: continue where the active-set kernel handed over (or do nothing)
  int first_sweep = 0;
  if (ctl != nullptr) {
    if (ctl[0] == 0) return;
    first_sweep = ctl[1];
  }
  const int m = 3 * nc;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  if (g0 != nullptr) {
    for (int i = tid; i < m; i += 1024) g[i] = g0[i];
  } else {
    for (int i = wv; i < m; i += 16) {
      double sacc = 0.0;
      for (int j = ln; j < m; j += 64) sacc = fma((double)W[(long)i * m + j], lam[j], sacc);
      for (int o = 32; o > 0; o >>= 1) sacc += __shfl_xor(sacc, o, 64);
      if (ln == 0) g[i] = d[i] + h2 * sacc;
    }
  }
  for (int c = tid; c < nc; c += 1024)
    nz[c] = (lam[3 * c] != 0.0 || lam[3 * c + 1] != 0.0 || lam[3 * c + 2] != 0.0) ? 1 : 0;
  if (tid == 0) stop = 0;
  __syncthreads();
  double dsum = 0.0;   // wave 0: sum of squared changes in this sweep
  int sweep = 0;
  double eps = 0.0;
  for (sweep = first_sweep; sweep < max_sweeps; ++sweep) {
    dsum = 0.0;
    int a = 0;
    while (true) {
      if (wv == 0) {
        int next = nc;
        while (a < nc) {
          const int c = a + ln;
          const bool active = (c < nc) && (nz[c] != 0 || g[3 * c] < 0.0);
          const unsigned long long bal = __ballot(active);
          if (bal == 0ull) {
            if (c < nc) status[c] = (int8_t)ICR_SEPARATE;
            a += 64;
            continue;
          }
          const int first = __ffsll((long long)bal) - 1;
          if (ln < first && c < nc) status[c] = (int8_t)ICR_SEPARATE;
          next = a + first;
          break;
        }
        if (next < nc) {
          // every lane of wave 0 runs the local solve on the same data
          double w[3][3], lo[3], dd[3];
          for (int i = 0; i < 3; ++i) {
            lo[i] = lam[3 * next + i];
            for (int j = 0; j < 3; ++j) w[i][j] = h2 * (double)W[(3L * next + i) * m + 3L * next + j];
          }
          for (int i = 0; i < 3; ++i)
            dd[i] = g[3 * next + i] - (w[i][0] * lo[0] + w[i][1] * lo[1] + w[i][2] * lo[2]);
          Local r = local_solve(w, dd, mu[next], j_inner);
          double dl[3];
          for (int i = 0; i < 3; ++i) {
            dl[i] = r.l[i] - lo[i];
            dsum += dl[i] * dl[i];
          }
          if (ln == 0) {
            for (int i = 0; i < 3; ++i) {
              bc[i] = dl[i];
              lam[3 * next + i] = r.l[i];
            }
            status[next] = (int8_t)r.st;
            nz[next] = (r.l[0] != 0.0 || r.l[1] != 0.0 || r.l[2] != 0.0) ? 1 : 0;
          }
        }
        if (ln == 0) ctl_s = next;
      }
      __syncthreads();
      const int cur = ctl_s;
      if (cur >= nc) break;
      const double d0 = bc[0], d1 = bc[1], d2 = bc[2];
      if (d0 != 0.0 || d1 != 0.0 || d2 != 0.0) {
        const TW *r0 = W + (3L * cur) * m;
        for (int i = tid; i < m; i += 1024)
          g[i] += h2 * ((double)r0[i] * d0 + (double)r0[m + i] * d1 + (double)r0[2L * m + i] * d2);
      }
      __syncthreads();
      a = cur + 1;
    }
    // eps = |lam_i - lam_{i-1}| / |lam_i|
    double part = 0.0;
    for (int i = tid; i < m; i += 1024) part += lam[i] * lam[i];
    __threadfence_block();
    double nl2 = block_sum(part, red);
    if (tid == 0) {
      double diff = sqrt(dsum), nl = sqrt(nl2);
      eps = nl > 0.0 ? diff / nl : (diff == 0.0 ? 0.0 : INFINITY);
      stop = (eps <= tol) ? 1 : 0;
    }
    __syncthreads();
    if (stop) {
      ++sweep;
      break;
    }
  }
  if (tid == 0) {
    *sweeps_out = sweep;
    *eps_out = eps;
  }
}

// Gauss-Seidel with the directions updated before every local solve (the
// per-constraint variant of the results section), one workgroup.  The current
// proximity P = p_free + h^2 W_H f of every contact (world frame) lives in
// LDS.  At contact a's turn: frame C_a and gap delta at P_a, block
// W~_aa = h^2 C_a W_H,aa C_a^T, gap without the own force
// d = delta - W~_aa C_a f_a (the linearisation of Algorithm 3 at P_a), local
// solve, f_a = C_a^T lambda_a, then P += h^2 W_H[:, a] (f_a - f_a^old) from
// the rows of the exactly symmetric W_H.  A contact with no force and a
// non-negative normal gap is a no-op; wave 0 finds the next contact that can
// change 64 at a time and writes the frames of the skipped ones.
__host__ __device__ inline size_t pgs_pc_lds(int nc) { return (size_t)nc * 3 * sizeof(double); }
__global__ __launch_bounds__(1024) void k_pgs_pc(int nc, const StepCtx *__restrict__ ctx,
                                                 const double *__restrict__ WH, const double *__restrict__ pin,
                                                 const double *__restrict__ pstart, const double *__restrict__ mu,
                                                 double h2, double *__restrict__ f, double *__restrict__ C,
                                                 double *__restrict__ lam, int8_t *__restrict__ status,
                                                 int max_sweeps, double tol, int j_inner, int *__restrict__ sweeps_out,
                                                 double *__restrict__ eps_out, const int *__restrict__ ctl) {
  // resume mode: continue where the register-chain kernel handed over (or
  // do nothing); pin then holds the proximity of the hand-over state
  int first_sweep = 0;
  if (ctl != nullptr) {
    if (ctl[0] == 0) return;
    first_sweep = ctl[1];
  }
  extern __shared__ double lds_P[];
  double *P = lds_P;
  __shared__ double bc[3];
  __shared__ double red[16];
  __shared__ int ctl_s;
  __shared__ int stop;
  const int m = 3 * nc;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const icr_obstacle obs = ctx->obs;
  const double t0 = ctx->t0, t1 = ctx->t0 + ctx->h;
  for (int i = tid; i < m; i += 1024) P[i] = pin[i];
  if (tid == 0) stop = 0;
  __syncthreads();
  int sweep = 0;
  double eps = 0.0, dsum = 0.0;
  for (sweep = first_sweep; sweep < max_sweeps; ++sweep) {
    dsum = 0.0;
    int a = 0;
    while (true) {
      if (wv == 0) {
        int next = nc;
        while (a < nc) {
          const int c = a + ln;
          bool active = false;
          double Fc[3][3], dc[3];
          if (c < nc) {
            const double pc[3] = {P[3 * c], P[3 * c + 1], P[3 * c + 2]};
            const double ps[3] = {pstart[3 * c], pstart[3 * c + 1], pstart[3 * c + 2]};
            contact_frame(obs, t0, t1, pc, ps, Fc, dc);
            active = f[3 * c] != 0.0 || f[3 * c + 1] != 0.0 || f[3 * c + 2] != 0.0 || dc[0] < 0.0;
          }
          const unsigned long long bal = __ballot(active);
          const int first = bal ? __ffsll((long long)bal) - 1 : 64;
          if (c < nc && ln < first) {   // skipped: separate, frame at its (unchanged) proximity
            for (int r = 0; r < 3; ++r) {
              for (int q = 0; q < 3; ++q) C[9L * c + 3 * r + q] = Fc[r][q];
              lam[3 * c + r] = 0.0;
            }
            status[c] = (int8_t)ICR_SEPARATE;
          }
          if (bal == 0ull) {
            a += 64;
            continue;
          }
          next = a + first;
          break;
        }
        if (next < nc) {
          // every lane of wave 0 runs the local solve on the same data
          const double pc[3] = {P[3 * next], P[3 * next + 1], P[3 * next + 2]};
          const double ps[3] = {pstart[3 * next], pstart[3 * next + 1], pstart[3 * next + 2]};
          double F[3][3], delta[3];
          contact_frame(obs, t0, t1, pc, ps, F, delta);
          double B[3][3];   // W_H,aa C_a^T
          for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) {
              const double *wr = WH + (3L * next + i) * m + 3L * next;
              B[i][j] = wr[0] * F[j][0] + wr[1] * F[j][1] + wr[2] * F[j][2];
            }
          double w[3][3];
          for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) w[i][j] = h2 * (F[i][0] * B[0][j] + F[i][1] * B[1][j] + F[i][2] * B[2][j]);
          for (int i = 0; i < 3; ++i)   // exactly symmetric block
            for (int j = 0; j < i; ++j) w[j][i] = w[i][j];
          const double fo[3] = {f[3 * next], f[3 * next + 1], f[3 * next + 2]};
          double lr[3], dd[3];
          for (int i = 0; i < 3; ++i) lr[i] = F[i][0] * fo[0] + F[i][1] * fo[1] + F[i][2] * fo[2];
          for (int i = 0; i < 3; ++i) dd[i] = delta[i] - (w[i][0] * lr[0] + w[i][1] * lr[1] + w[i][2] * lr[2]);
          const PgsRec rec = make_record(w, mu[next]);
          const Local r =
              j_inner == 8 ? local_solve_rec<8>(rec, dd, j_inner) : local_solve_rec<0>(rec, dd, j_inner);
          double fn[3], df[3];
          for (int q = 0; q < 3; ++q) {
            fn[q] = F[0][q] * r.l[0] + F[1][q] * r.l[1] + F[2][q] * r.l[2];
            df[q] = fn[q] - fo[q];
            dsum += df[q] * df[q];
          }
          if (ln == 0) {
            for (int q = 0; q < 3; ++q) {
              bc[q] = df[q];
              f[3 * next + q] = fn[q];
              lam[3 * next + q] = r.l[q];
              for (int k = 0; k < 3; ++k) C[9L * next + 3 * q + k] = F[q][k];
            }
            status[next] = (int8_t)r.st;
          }
        }
        if (ln == 0) ctl_s = next;
      }
      __syncthreads();
      const int cur = ctl_s;
      if (cur >= nc) break;
      const double d0 = bc[0], d1 = bc[1], d2 = bc[2];
      if (d0 != 0.0 || d1 != 0.0 || d2 != 0.0) {
        const double *r0 = WH + (3L * cur) * m;
        for (int i = tid; i < m; i += 1024) P[i] += h2 * (r0[i] * d0 + r0[m + i] * d1 + r0[2L * m + i] * d2);
      }
      __syncthreads();
      a = cur + 1;
    }
    // eps = |f_i - f_{i-1}| / |f_i|
    double part = 0.0;
    __threadfence_block();
    for (int i = tid; i < m; i += 1024) part += f[i] * f[i];
    const double nf2 = block_sum(part, red);
    if (tid == 0) {
      const double diff = sqrt(dsum), nf = sqrt(nf2);
      eps = nf > 0.0 ? diff / nf : (diff == 0.0 ? 0.0 : INFINITY);
      stop = (eps <= tol) ? 1 : 0;
    }
    __syncthreads();
    if (stop) {
      ++sweep;
      break;
    }
  }
  if (tid == 0) {
    *sweeps_out = sweep;
    *eps_out = eps;
  }
}

// Active-set projected Gauss-Seidel (exact).  In a sweep only contacts with
// a non-zero force or a negative gap can change; all others are no-ops of
// Gauss-Seidel.  The kernel keeps the set S of contacts that may change and
// runs the sequential sweep over S alone, with the compact coupling block
// W~_SS (gathered once per set) and per-contact records (3x3 block, its
// inverse, mu) in LDS.  The sweep is a barrier-free chain over gaps and
// forces in registers, of one wave for every 64 contacts (chain_sweep).  It
// then verifies that every contact outside S was a no-op at its turn, i.e.
// that its normal gap
//   g_n(c) = g_n^set(c) + W~_{n(c),S} (lambda^turn - lambda^set) >= 0,
// with lambda^turn the force of S contacts before c in this sweep and after c
// from the previous sweep.  Cauchy-Schwarz on the PSD matrix W~ bounds the
// correction by sqrt(W~_cc) * sum_q sqrt(W~_qq) |lambda^turn_q - lambda^set_q|,
// which settles almost every contact; the others are evaluated exactly, and
// once as many have been as are skipped, all are and the sweep's end becomes
// the reference state, from which the changes shrink as the sweeps converge.
// (With the set's start as the only reference a warm start some way off left
// the same contacts unsettled in every sweep: 1000 contacts of which 12 % are
// pressed took 330 us a sweep, the chain of those 42; 30 sweeps 10.1 ms, now
// 2.6.)  On a violation the violating contacts join S and the sweep restarts
// from its start state, so the iterates are those of the full sequential
// sweep.  If S outgrows PGS_SMAX the remaining sweeps go to k_pgs_single (ctl[0] = 1).
constexpr int PGS_SMAX = 512;
constexpr int PGS_S3 = 3 * PGS_SMAX;
constexpr int PGS_NT = 512;   // threads of the active-set kernel
constexpr int PGS_NW = PGS_NT / 64;
constexpr int PGS_WAVE_MAX = kPgsWaveMax;   // largest set swept by the register chains (= PGS_SMAX)
constexpr int PGS_BLK = kPgsBlk;            // doubles per 3x3 block of the blocked W~_SS
struct PgsLds {
  // gaps without the own term, current forces (written by the running sweep),
  // forces at the sweep's start and at the set's
  double gS[PGS_S3], lamS[PGS_S3], lamS0[PGS_S3], lamSet[PGS_S3];
  double rec[PGS_RW * PGS_SMAX];   // row q of contact i at q PGS_SMAX + i (see pgs_rec_load)
  double red[48];
  int Sidx[PGS_SMAX];
  unsigned char stS[PGS_SMAX];
  int wcount[64];
  unsigned short ulist[PGS_MAX_NC];
  unsigned char inS[PGS_MAX_NC];
  double Rmin;   // settle threshold of the set: B below it settles every skipped contact
  int nS, flag, stop, nu, zflag;
  int cprog, cflag;   // contacts solved by the chain (counted on over the sweeps); block Gauss-Seidel: next block staged
  int perr;           // a wait of the ring sweep ran out
};

static_assert(sizeof(PgsLds) <= 160 * 1024, "active-set PGS state must fit one CU's LDS");
static_assert(3 * PGS_MAX_NC * sizeof(double) + PGS_MAX_NC + 512 <= 160 * 1024, "k_pgs_single LDS");


__device__ inline double readlane_f64(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Blocked couplings of a set padded to nsp contacts (a multiple of 64): the
// 3x3 block (rows of contact c, columns of contact i) of column i lies in the
// group of 64 rows c / 64, 576 doubles each, entry j (row-major) of lane
// l = c % 64 at blk_entry(l, j): pairs of entries lane by lane, so that each
// of a wave's five loads of a column's group is contiguous.  (With the nine
// doubles of a lane side by side every load touched all 40 cache lines of the
// group, which cost sets of several waves a third of their time.)
constexpr int BLK_GROUP = kPgsGroup;
__host__ __device__ constexpr inline int blk_entry(int l, int j) {
  return j < 8 ? 128 * (j / 2) + 2 * l + (j & 1) : 512 + l;
}
// entry r of a group, 0 <= r < BLK_GROUP -> lane and block entry
__device__ inline void blk_index(int r, int &l, int &j) {
  l = r < 512 ? (r & 127) >> 1 : r - 512;
  j = r < 512 ? 2 * (r >> 7) + (r & 1) : 8;
}
struct BlkCol {
  double2 x[4];
  double y;
};
// A buffer of blocked couplings: column groups are read with the column's
// byte offset in a scalar register and per-lane constants in vector
// registers, so a load needs no address arithmetic.  The scalar offset is not
// range checked: it has to be that of a column (PgsColumns).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
struct BlkBuf {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ __forceinline__ BlkBuf(const double *p, unsigned bytes)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, bytes, 0x00027000)) {}
};
// off: byte offset of the column's group (uniform)
__device__ __forceinline__ void blk_load(BlkCol &X, const BlkBuf &b, unsigned off, int ln) {
  const unsigned o = 16u * (unsigned)ln, o8 = 4096u + 8u * (unsigned)ln;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    X.x[k] = __builtin_bit_cast(double2, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(b.rsrc, o + 1024u * k, off, 0));
  X.y = __builtin_bit_cast(double, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(b.rsrc, o8, off, 0));
}
// e += block * (d0, d1, d2)
__device__ __forceinline__ void blk_apply(double (&e)[3], const BlkCol &X, double d0, double d1, double d2) {
  e[0] = fma(X.x[1].x, d2, fma(X.x[0].y, d1, fma(X.x[0].x, d0, e[0])));
  e[1] = fma(X.x[2].y, d2, fma(X.x[2].x, d1, fma(X.x[1].y, d0, e[1])));
  e[2] = fma(X.y, d2, fma(X.x[3].y, d1, fma(X.x[3].x, d0, e[2])));
}
// Columns of a group in flight ahead of the one in use.  A stick visit takes
// 0.17 us, an L2 hit 0.07 us and a miss 0.35 us; two columns were as fast as
// four on sets that stay in L2, eight no faster.
constexpr int PGS_AHEAD = kPgsAhead;

// The chain's state of one contact, in one lane's registers.
struct ChainLane {
  PgsRec rc;
  double e[3], l[3];   // gap without the own term, force
  int st;
};
__device__ __forceinline__ PgsRec pgs_rec_load(const PgsLds &L, int c) {
  PgsRec r;
  double *x = reinterpret_cast<double *>(&r);
#pragma unroll
  for (int q = 0; q < PGS_RC; ++q) x[q] = L.rec[q * PGS_SMAX + c];
  return r;
}

// One Gauss-Seidel visit: the contact of lane li, whose own lane holds its
// record, force and gap without the own term e = g - W~_cc lambda_c (the
// blocked W~ has zero diagonal blocks, so the update keeps it exact).  The
// force change is broadcast through scalar registers and every lane applies
// W~(own rows, contact) to its gap.  Nothing is read from LDS; lane li stores
// its new force to L.lamS and, with PUB (another wave follows), then the count
// of solved contacts, which each lane holds in `prog`, to L.cprog (LDS
// operations of one wave complete in order, so a reader that sees the count
// sees the force; the compiler fence keeps the stores in that order).  A wave
// runs every instruction for all lanes and pays for each 4 to 6 cycles, so
// what counts is their number and size: a visit has two branches, each on one
// bit of a mask, and lane li's stores and the broadcast share one change of
// the execution mask (a v_readlane with the lane in a scalar register takes
// 9.5 cycles, the v_readfirstlane of the only active lane 5.5).  A stick visit
// takes 410 cycles, a slip visit 1090, a visit that ends at once 130.  With
// the record read from LDS, the solve repeated on broadcast data and the
// normalised passes, a visit of half sticking, half slipping contacts took
// 425 ns in a set of 64 contacts and 621 in one of 512; now 322 and 367.
// nz: lanes whose contact carried a force at the sweep's start; a contact
// without one whose gap is not negative stays as it is, and its visit ends at
// once.  safe: lanes whose record allows the fast slip passes.  slip: lanes
// that slipped.  open: lanes with a gap that is not negative, taken at the end
// of the last visit.
struct ChainMasks {
  unsigned long long nz, safe, slip, open;
};
__device__ __forceinline__ unsigned lds_addr(const void *p) {
  return (unsigned)(unsigned long long)(__attribute__((address_space(3))) const void *)p;
}
// l to L.lamS (its byte address in at) and, with PUB, prog to L.cprog (pat), from
// the lane of `bit`; its change d as uniform values.  All lanes are active.
template <bool PUB>
__device__ __forceinline__ void chain_commit(double l0, double l1, double l2, double (&d)[3], unsigned at,
                                             unsigned pat, int prog, unsigned long long bit) {
  unsigned s0, s1, s2, s3, s4, s5;
  const unsigned long long x0 = __builtin_bit_cast(unsigned long long, d[0]),
                           x1 = __builtin_bit_cast(unsigned long long, d[1]),
                           x2 = __builtin_bit_cast(unsigned long long, d[2]);
#define ICR_RFL6                     \
  "v_readfirstlane_b32 %0, %7\n\t"   \
  "v_readfirstlane_b32 %1, %8\n\t"   \
  "v_readfirstlane_b32 %2, %9\n\t"   \
  "v_readfirstlane_b32 %3, %10\n\t"  \
  "v_readfirstlane_b32 %4, %11\n\t"  \
  "v_readfirstlane_b32 %5, %12\n\t"  \
  "s_mov_b64 exec, -1"
#define ICR_RFL6_OPS                                                                                          \
  "=&s"(s0), "=&s"(s1), "=&s"(s2), "=&s"(s3), "=&s"(s4), "=&s"(s5)                                            \
      : "s"(bit), "v"((unsigned)x0), "v"((unsigned)(x0 >> 32)), "v"((unsigned)x1), "v"((unsigned)(x1 >> 32)), \
        "v"((unsigned)x2), "v"((unsigned)(x2 >> 32)), "v"(at), "v"(l0), "v"(l1), "v"(l2)
  if constexpr (PUB)
    asm volatile(
        "s_mov_b64 exec, %6\n\t"
        "ds_write2_b64 %13, %14, %15 offset1:1\n\t"
        "ds_write_b64 %13, %16 offset:16\n\t"
        "ds_write_b32 %17, %18\n\t" ICR_RFL6
        : ICR_RFL6_OPS, "v"(pat), "v"(prog)
        : "memory");
  else
    asm volatile(
        "s_mov_b64 exec, %6\n\t"
        "ds_write2_b64 %13, %14, %15 offset1:1\n\t"
        "ds_write_b64 %13, %16 offset:16\n\t" ICR_RFL6
        : ICR_RFL6_OPS
        : "memory");
#undef ICR_RFL6
#undef ICR_RFL6_OPS
  d[0] = __builtin_bit_cast(double, (unsigned long long)s1 << 32 | s0);
  d[1] = __builtin_bit_cast(double, (unsigned long long)s3 << 32 | s2);
  d[2] = __builtin_bit_cast(double, (unsigned long long)s5 << 32 | s4);
}
// e += X d for uniform d, in place (left to itself, the compiler moves e to new
// registers and back around the branch of the visit).
__device__ __forceinline__ void blk_apply_uniform(double (&e)[3], const BlkCol &X, const double (&d)[3]) {
  asm("v_fmac_f64_e32 %0, %3, %6\n\t"
      "v_fmac_f64_e32 %1, %3, %9\n\t"
      "v_fmac_f64_e32 %2, %3, %12\n\t"
      "v_fmac_f64_e32 %0, %4, %7\n\t"
      "v_fmac_f64_e32 %1, %4, %10\n\t"
      "v_fmac_f64_e32 %2, %4, %13\n\t"
      "v_fmac_f64_e32 %0, %5, %8\n\t"
      "v_fmac_f64_e32 %1, %5, %11\n\t"
      "v_fmac_f64_e32 %2, %5, %14"
      : "+v"(e[0]), "+v"(e[1]), "+v"(e[2])
      : "s"(d[0]), "s"(d[1]), "s"(d[2]), "v"(X.x[0].x), "v"(X.x[0].y), "v"(X.x[1].x), "v"(X.x[1].y), "v"(X.x[2].x),
        "v"(X.x[2].y), "v"(X.x[3].x), "v"(X.x[3].y), "v"(X.y));
}
template <int J, bool PUB>
__device__ __forceinline__ void chain_visit(ChainLane &c, const BlkCol &X, int li, unsigned at, unsigned pat, int prog,
                                            int j_inner, ChainMasks &k) {
  const unsigned long long bit = 1ull << li;
  if (lane_in(~k.open | k.nz, bit)) {
    const Trial t = stick_trial(c.rc, c.e[0], c.e[1], c.e[2]);
    double l[3] = {t.ln, t.lt1, t.lt2};
    if (!lane_in(t.stick & ~k.open, bit)) {
      if (!lane_in(k.open, bit)) {
        slip_solve<J>(c.rc, t, c.e[0], c.e[1], c.e[2], j_inner, bit, k.safe, l);
        k.slip |= bit;
      } else {
        l[0] = l[1] = l[2] = 0.0;
      }
    }
    double d[3] = {l[0] - c.l[0], l[1] - c.l[1], l[2] - c.l[2]};
    chain_commit<PUB>(l[0], l[1], l[2], d, at, pat, prog, bit);
    blk_apply_uniform(c.e, X, d);
  }
}

// The n contacts of this wave's lanes 0 .. n-1 in order (and, up to a
// multiple of PGS_AHEAD, lanes beyond them, whose gap and force are zero);
// cols: their columns' groups of this wave's rows.  prog: the count of solved contacts after this lane's.
template <int J, bool PUB>
__device__ __forceinline__ void chain_solve(ChainLane &c, int n, const BlkBuf &B, PgsColumns cols, int me, int prog,
                                            PgsLds &L, int j_inner, int ln) {
  ChainMasks k{__ballot((c.l[0] != 0.0) | (c.l[1] != 0.0) | (c.l[2] != 0.0)), __ballot(c.rc.it00 > 0.0), 0ull,
               __ballot(c.e[0] >= 0.0)};
  const unsigned at = lds_addr(L.lamS + 3 * me), pat = lds_addr(&L.cprog);
  BlkCol X[PGS_AHEAD];
#pragma unroll
  for (int u = 0; u < PGS_AHEAD; ++u) {
    blk_load(X[u], B, cols.take(), ln);
    __builtin_amdgcn_sched_barrier(0);   // in column order: the first use waits for the first column only
  }
  for (int i = 0; i < n; i += PGS_AHEAD) {
#pragma unroll
    for (int u = 0; u < PGS_AHEAD; ++u) {
      chain_visit<J, PUB>(c, X[u], i + u, at, pat, prog, j_inner, k);
      // the mask of the comparison is ready behind the loads
      k.open = __ballot(c.e[0] >= 0.0);
      __builtin_amdgcn_sched_barrier(0);
      blk_load(X[u], B, cols.take(), ln);
    }
  }
  // Visits that ended at once have published nothing: the whole count.  The
  // last visit may have published it, and then the next wave may be past it:
  // the count never goes back.
  if (PUB && ln == n - 1) __hip_atomic_fetch_max(&L.cprog, prog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  // a contact that sticks has a positive normal force
  c.st = ((k.slip >> ln) & 1ull) ? ICR_SLIP : L.lamS[3 * (ln < n ? me : me - ln)] != 0.0 ? ICR_STICK : ICR_SEPARATE;
}

// A set of up to 512 contacts is swept by R = ceil(nS / 64) waves: wave w
// keeps the gaps of contacts 64 w .. 64 w + 63.  The contacts are solved in
// order, each 64-contact block by the wave that keeps its gaps, while every
// other wave applies each force change to its own gaps as soon as it is
// published; no wave applies another block's updates on the solving chain,
// and no barrier is taken.  Every gap receives the same products in the same
// order as in a one-wave sweep.  A wave solves its block only after it has
// applied every earlier block, so each wait is on a wave that is making
// progress.  A wait that runs out (a broken count, not an input) sets L.perr.
constexpr int RING_SPIN = 1 << 24;
__device__ __forceinline__ void ring_wait(PgsLds &L, int prog, int &seen) {
  if (seen >= prog) return;
  for (int spin = 0;; ++spin) {
    seen = __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(&L.cprog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    if (seen >= prog) break;
    if (spin == RING_SPIN) {
      __hip_atomic_store(&L.perr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      break;
    }
    if ((spin & 255) == 255 && __hip_atomic_load(&L.perr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0)
      break;   // another wave already gave up: no more waiting in this sweep
    __builtin_amdgcn_s_sleep(1);
  }
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
// The applying part: the changes of contacts b .. b + n - 1 of the LDS arrays,
// solved by another wave, added to this wave's gaps in contact order.  prog0:
// the count before the first one.
__device__ __forceinline__ void ring_apply(ChainLane &c, int n, const BlkBuf &B, PgsColumns cols, int b, int prog0,
                                           PgsLds &L, int ln) {
  BlkCol X[PGS_AHEAD];
#pragma unroll
  for (int u = 0; u < PGS_AHEAD; ++u) {
    blk_load(X[u], B, cols.take(), ln);
    __builtin_amdgcn_sched_barrier(0);
  }
  int seen = prog0;
  for (int i = 0; i < n; i += PGS_AHEAD) {
#pragma unroll
    for (int u = 0; u < PGS_AHEAD; ++u) {
      if (i + u < n) {
        ring_wait(L, prog0 + i + u + 1, seen);
        const double *l = L.lamS + 3 * (b + i + u), *l0 = L.lamS0 + 3 * (b + i + u);
        blk_apply(c.e, X[u], l[0] - l0[0], l[1] - l0[1], l[2] - l0[2]);
        blk_load(X[u], B, cols.take(), ln);
      }
    }
  }
}

// One sweep over nS contacts, padded to nsp, by wave w < nsp / 64; o: first
// contact of the set in the LDS arrays (L.lamS = L.lamS0 = the forces at the
// sweep's start), prog0: the count of solved contacts before the sweep, which
// adds nsp.
template <int J, bool PUB>
__device__ __forceinline__ void chain_sweep(ChainLane &c, int nS, int nsp, const BlkBuf &B, int o, int prog0,
                                            PgsLds &L, int j_inner, int w, int ln) {
  const unsigned stride = 8u * PGS_BLK * (unsigned)nsp, col = 8u * BLK_GROUP * (unsigned)w;
  const int me = o + 64 * w + ln, prog = prog0 + 64 * w + ln + 1;
  if (!PUB) {
    chain_solve<J, false>(c, nS, B, PgsColumns(col, stride, nS), me, prog, L, j_inner, ln);
    return;
  }
  for (int b = 0; b < nS; b += 64) {
    const int n = min(64, nS - b);
    const PgsColumns cols(col + stride * (unsigned)b, stride, n);
    if (b == 64 * w) {
      __builtin_amdgcn_s_setprio(3);   // the solving wave first on its SIMD
      chain_solve<J, true>(c, n, B, cols, me, prog, L, j_inner, ln);
      __builtin_amdgcn_s_setprio(0);
    } else {
      ring_apply(c, n, B, cols, o + b, prog0 + b, L, ln);
    }
  }
}

// The active set of the first sweep, its compact couplings and records are
// prepared by a wide kernel before the sequential kernel starts (a set that
// grows later is rebuilt inside k_pgs_active).
// Entry e of the blocked couplings of the set Sidx (nS contacts padded to
// nsp): h^2 W of the block, zero diagonal blocks and padding.  The rows of
// contact i stand for its columns (W is exactly symmetric), so consecutive
// lanes read neighbouring columns of one row.
template <class TW>
__device__ __forceinline__ double blk_value(long e, int nS, int nsp, const int *Sidx, const TW *__restrict__ W, int m,
                                            double h2) {
  const int per = nsp * PGS_BLK;
  const int i = (int)(e / per), r = (int)(e % per);
  int l, j;
  blk_index(r % BLK_GROUP, l, j);
  const int c = 64 * (r / BLK_GROUP) + l;
  if (c >= nS || c == i) return 0.0;
  return h2 * (double)W[(3L * Sidx[i] + j % 3) * m + 3L * Sidx[c] + j / 3];
}

// k_pgs_gather (any grid): the normal gaps at the set's start and sqrt(W~_nn)
// of every contact; every block forms the set S = {c : lambda_c != 0 or
// g0_n(c) < 0} in ascending order (64-contact ballots, window prefix) and
// block 0 writes S and |S|.  For a set of at most PGS_WAVE_MAX contacts the blocks then
// write the blocked W~_SS with zero diagonal blocks, the per-contact records
// (row q of contact i at q |S| + i: PgsRec, then the square roots of the
// block's diagonal) and the gaps without the own term, e = g0 - W~_cc lambda_c.
template <class TW>
__device__ __forceinline__ void pgs_gather(int nc, const TW *__restrict__ W, const double *__restrict__ g0,
                                           const double *__restrict__ lam, const double *__restrict__ mu, double h2,
                                           int *__restrict__ Sidx_out, int *__restrict__ nS_out,
                                           double *__restrict__ gnSet, double *__restrict__ swn,
                                           double *__restrict__ Wss, double *__restrict__ rec,
                                           double *__restrict__ gS) {
  __shared__ int Sidx[PGS_MAX_NC];
  __shared__ int wcount[PGS_MAX_NC / 64 + 1];
  __shared__ int nS_s;
  const int m = 3 * nc;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const int nwin = (nc + 63) / 64;
  const long stride = (long)gridDim.x * blockDim.x, t0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long c = t0; c < nc; c += stride) {
    gnSet[c] = g0[3 * c];
    swn[c] = sqrt(h2 * (double)W[(3L * c) * m + 3L * c]);
  }
  auto in_set = [&](int c) {
    return c < nc && (lam[3 * c] != 0.0 || lam[3 * c + 1] != 0.0 || lam[3 * c + 2] != 0.0 || g0[3 * c] < 0.0);
  };
  for (int w = wv; w < nwin; w += 4) {
    const unsigned long long bal = __ballot(in_set(64 * w + ln));
    if (ln == 0) wcount[w] = __popcll(bal);
  }
  __syncthreads();
  if (tid == 0) {
    int acc = 0;
    for (int w = 0; w < nwin; ++w) {
      const int t = wcount[w];
      wcount[w] = acc;
      acc += t;
    }
    nS_s = acc;
  }
  __syncthreads();
  for (int w = wv; w < nwin; w += 4) {
    const int c = 64 * w + ln;
    const bool in = in_set(c);
    const unsigned long long bal = __ballot(in);
    if (in) Sidx[wcount[w] + __popcll(bal & ((1ull << ln) - 1ull))] = c;
  }
  __syncthreads();
  const int nS = nS_s;
  if (blockIdx.x == 0) {
    for (int q = tid; q < nS; q += 256) Sidx_out[q] = Sidx[q];
    if (tid == 0) *nS_out = nS;
  }
  if (nS == 0 || nS > PGS_WAVE_MAX) return;
  const int nsp = pgs_wave_pad(nS);
  const long nel = (long)nS * nsp * PGS_BLK;
  for (long e = t0; e < nel; e += stride) Wss[e] = blk_value(e, nS, nsp, Sidx, W, m, h2);
  for (long i = t0; i < nS; i += stride) {
    double wb[3][3];
    const long ci = 3L * Sidx[i];
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) wb[p][q] = h2 * (double)W[(ci + p) * m + ci + q];
    const PgsRec tmp = make_record(wb, mu[Sidx[i]]);
    const double *x = reinterpret_cast<const double *>(&tmp);
    for (int q = 0; q < PGS_RC; ++q) rec[(long)q * nS + i] = x[q];
    for (int q = 0; q < 3; ++q) rec[(long)(PGS_RC + q) * nS + i] = sqrt(wb[q][q]);
  }
  for (long r = t0; r < 3L * nS; r += stride) {
    const long cr = 3L * Sidx[r / 3];
    const int a = (int)(r % 3);
    double own = 0.0;
    for (int q = 0; q < 3; ++q) own = fma(h2 * (double)W[(cr + a) * m + cr + q], lam[cr + q], own);
    gS[r] = g0[cr + a] - own;
  }
}
template <class TW>
__global__ __launch_bounds__(256) void k_pgs_gather(int nc, const TW *__restrict__ W,
                                                    const double *__restrict__ g0, const double *__restrict__ lam,
                                                    const double *__restrict__ mu, double h2,
                                                    int *__restrict__ Sidx_out, int *__restrict__ nS_out,
                                                    double *__restrict__ gnSet, double *__restrict__ swn,
                                                    double *__restrict__ Wss, double *__restrict__ rec,
                                                    double *__restrict__ gS) {
  pgs_gather<TW>(nc, W, g0, lam, mu, h2, Sidx_out, nS_out, gnSet, swn, Wss, rec, gS);
}

// The sequential kernel's body, for one workgroup of PGS_NT threads with the
// state L in its LDS (k_pgs_active, and each scene's workgroup of the batched
// Newton loops).  npre: size of the set prepared by pgs_gather (preSidx,
// preRec, preGS); a value above PGS_WAVE_MAX builds the first set here, from
// g0, gnSet and swn (a set too large for the chains is handed over).
template <class TW>
__device__ __forceinline__ void pgs_active_body(PgsLds &L, int nc, const TW *__restrict__ W,
                                                const double *__restrict__ d, const double *__restrict__ g0,
                                                const double *__restrict__ mu, double h2, double *__restrict__ lam,
                                                int8_t *__restrict__ status, int max_sweeps, double tol,
                                                int j_inner, int *__restrict__ sweeps_out,
                                                double *__restrict__ eps_out, double *__restrict__ Wss,
                                                double *__restrict__ gnSet, const double *__restrict__ swn,
                                                int *__restrict__ ctl, const int *__restrict__ preSidx, int npre,
                                                const double *__restrict__ preRec, const double *__restrict__ preGS) {
  const int m = 3 * nc;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  for (int c = tid; c < nc; c += PGS_NT) {
    bool nzc = lam[3 * c] != 0.0 || lam[3 * c + 1] != 0.0 || lam[3 * c + 2] != 0.0;
    L.inS[c] = (nzc || g0[3 * c] < 0.0) ? 1 : 0;
  }
  if (tid == 0) {
    L.zflag = 0;
    L.perr = 0;
    L.cprog = 0;
    ctl[0] = 0;
    ctl[1] = 0;
  }
  __syncthreads();
  const int wu = __builtin_amdgcn_readfirstlane(wv);
  int sweep = 0, nS = 0, ldS = 0, nsp = 0;
  int nsweep = 0, prog = 0;   // sweeps run and contacts solved, restarted sweeps included
  int nexact = 0;             // gaps evaluated exactly since the reference state was set
  double eps = 0.0;
  bool need_build = true, first_build = true, built = false;
  while (sweep < max_sweeps) {
    if (need_build && first_build && npre <= PGS_WAVE_MAX) {
      // ---- the prepared first set: copy it in
      nS = __builtin_amdgcn_readfirstlane(npre);
      ldS = 3 * nS;
      nsp = pgs_wave_pad(nS);
      for (int i = tid; i < nS; i += PGS_NT) L.Sidx[i] = preSidx[i];
      for (int e = tid; e < nS * (PGS_RC + 3); e += PGS_NT) L.rec[PGS_SMAX * (e / nS) + e % nS] = preRec[e];
      for (int r = tid; r < ldS; r += PGS_NT) L.gS[r] = preGS[r];
      __syncthreads();
      for (int r = tid; r < ldS; r += PGS_NT) {
        L.lamS[r] = lam[3 * L.Sidx[r / 3] + r % 3];
        L.lamSet[r] = L.lamS[r];
      }
      __syncthreads();
      need_build = false;
      first_build = false;
      built = true;
    }
    if (need_build) {
      // ---- ordered list of S (ballot per 64-contact window, prefix by thread 0)
      const int nwin = (nc + 63) / 64;
      for (int w = wv; w < nwin; w += PGS_NW) {
        const int c = 64 * w + ln;
        const unsigned long long bal = __ballot(c < nc && L.inS[c]);
        if (ln == 0) L.wcount[w] = __popcll(bal);
      }
      __syncthreads();
      if (tid == 0) {
        int acc = 0;
        for (int w = 0; w < nwin; ++w) {
          int t = L.wcount[w];
          L.wcount[w] = acc;
          acc += t;
        }
        L.nS = acc;
      }
      __syncthreads();
      nS = __builtin_amdgcn_readfirstlane(L.nS);
      if (nS > PGS_SMAX) {   // hand over: global lambda holds the sweep-start state
        if (tid == 0) {
          ctl[0] = 1;
          ctl[1] = sweep;
        }
        return;
      }
      for (int w = wv; w < nwin; w += PGS_NW) {
        const int c = 64 * w + ln;
        const bool in = c < nc && L.inS[c];
        const unsigned long long bal = __ballot(in);
        if (in) L.Sidx[L.wcount[w] + __popcll(bal & ((1ull << ln) - 1ull))] = c;
      }
      __syncthreads();
      ldS = 3 * nS;
      nsp = pgs_wave_pad(nS);
      for (int r = tid; r < ldS; r += PGS_NT) {
        L.lamS[r] = lam[3 * L.Sidx[r / 3] + r % 3];
        L.lamSet[r] = L.lamS[r];
      }
      // ---- compact couplings W~_SS (padded to nsp contacts) and records
      {
        const long nel = (long)nS * nsp * PGS_BLK;
        for (long e = tid; e < nel; e += PGS_NT) Wss[e] = blk_value(e, nS, nsp, L.Sidx, W, m, h2);
      }
      __threadfence_block();
      __syncthreads();
      for (int i = tid; i < nS; i += PGS_NT) {
        double wb[3][3];
        const long ci = 3L * L.Sidx[i];
        for (int p = 0; p < 3; ++p)
          for (int q = 0; q < 3; ++q) wb[p][q] = h2 * (double)W[(ci + p) * m + ci + q];
        const PgsRec tmp = make_record(wb, mu[L.Sidx[i]]);
        const double *x = reinterpret_cast<const double *>(&tmp);
        for (int q = 0; q < PGS_RC; ++q) L.rec[q * PGS_SMAX + i] = x[q];
        for (int q = 0; q < 3; ++q) L.rec[(PGS_RC + q) * PGS_SMAX + i] = sqrt(wb[q][q]);
      }
      // ---- gaps at the set's start state (lambda is zero outside S)
      if (first_build) {
        // g0 = d + W~ lambda0 was formed by k_sym_gemv_sparse for every row; the
        // chains keep the gap without the contact's own term
        for (int r = tid; r < ldS; r += PGS_NT) {
          const long cr = 3L * L.Sidx[r / 3];
          double own = 0.0;
          for (int q = 0; q < 3; ++q) own = fma(h2 * (double)W[(cr + r % 3) * m + cr + q], L.lamS[r - r % 3 + q], own);
          L.gS[r] = g0[cr + r % 3] - own;
        }
      } else {
        for (int c = wv; c < nS; c += PGS_NW) {
          double a0 = 0.0, a1 = 0.0, a2 = 0.0;
          for (int i = ln; i < nS; i += 64) {
            const double *g = Wss + (long)i * nsp * PGS_BLK + (long)BLK_GROUP * (c / 64);
            double b[9];
#pragma unroll
            for (int j = 0; j < 9; ++j) b[j] = g[blk_entry(c % 64, j)];
            const double l0 = L.lamS[3 * i], l1 = L.lamS[3 * i + 1], l2 = L.lamS[3 * i + 2];
            a0 += b[0] * l0 + b[1] * l1 + b[2] * l2;
            a1 += b[3] * l0 + b[4] * l1 + b[5] * l2;
            a2 += b[6] * l0 + b[7] * l1 + b[8] * l2;
          }
          for (int o = 32; o > 0; o >>= 1) {
            a0 += __shfl_xor(a0, o, 64);
            a1 += __shfl_xor(a1, o, 64);
            a2 += __shfl_xor(a2, o, 64);
          }
          if (ln == 0) {
            const int cc = 3 * L.Sidx[c];
            L.gS[3 * c] = d[cc] + a0;
            L.gS[3 * c + 1] = d[cc + 1] + a1;
            L.gS[3 * c + 2] = d[cc + 2] + a2;
          }
        }
        for (int c = wv; c < nc; c += PGS_NW) {
          if (L.inS[c]) continue;
          double a = 0.0;
          for (int q = ln; q < ldS; q += 64)
            a = fma(h2 * (double)W[(3L * c) * m + 3L * L.Sidx[q / 3] + q % 3], L.lamS[q], a);
          for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
          if (ln == 0) gnSet[c] = d[3 * c] + a;
        }
      }
      __syncthreads();
      need_build = false;
      first_build = false;
      built = true;
    }
    if (built) {
      // Settle threshold of the new set.  A skipped contact c is settled when
      // g - sqrt(W~_cc) B > 1e-13 (|g| + sqrt(W~_cc) B), i.e. (sqrt(W~_cc) > 0)
      // B < (g - 1e-13 |g|) / (sqrt(W~_cc) (1 + 1e-13)); Rmin is the smallest
      // of these bounds, shrunk by 1e-12 for rounding, so B < Rmin settles
      // all of them at once (else the per-contact test runs).
      double rmin = INFINITY;
      int zf = 0;
      for (int c = tid; c < nc; c += PGS_NT) {
        if (L.inS[c]) continue;
        const double g = gnSet[c], w = swn[c];
        if (w > 0.0)
          rmin = fmin(rmin, (g - 1e-13 * fabs(g)) / (w * (1.0 + 1e-13)));
        else if (!(g > 0.0))
          zf = 1;
        status[c] = (int8_t)ICR_SEPARATE;
      }
      if (zf) atomicOr(&L.zflag, 1);
      const double rm = block_min(rmin, L.red);
      if (tid == 0) L.Rmin = rm > 0.0 ? rm * (1.0 - 1e-12) : rm * (1.0 + 1e-12);
      __syncthreads();
      built = false;
    }
    // ---- sweep over S from its start state, by the waves that hold its
    // contacts, and their part of the sweep's sums: squared changes,
    // |lambda|^2, and the bound factor of the skipped contacts' gaps
    // B = sum_q sqrt(W~_qq) max(|lamS - lamSet|, |lamS0 - lamSet|)
    double *red = L.red + 24 * (nsweep & 1);   // double-buffered: one barrier per sweep
    if (64 * wu < nS) {
      const int me = 64 * wu + ln;
      const bool on = me < nS;
      const BlkBuf buf(Wss, 8u * PGS_BLK * (unsigned)nsp * (unsigned)nS);
      ChainLane c;
      c.rc = pgs_rec_load(L, on ? me : 0);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        c.e[q] = on ? L.gS[3 * me + q] : 0.0;
        c.l[q] = on ? L.lamS[3 * me + q] : 0.0;
        if (on) L.lamS0[3 * me + q] = c.l[q];
      }
      if (nS <= 64) {
        if (j_inner == 8)
          chain_sweep<8, false>(c, nS, nsp, buf, 0, prog, L, j_inner, 0, ln);
        else
          chain_sweep<0, false>(c, nS, nsp, buf, 0, prog, L, j_inner, 0, ln);
      } else {
        if (j_inner == 8)
          chain_sweep<8, true>(c, nS, nsp, buf, 0, prog, L, j_inner, wu, ln);
        else
          chain_sweep<0, true>(c, nS, nsp, buf, 0, prog, L, j_inner, wu, ln);
      }
      double dpart = 0.0, bpart = 0.0, npart = 0.0;
      if (on) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const double ls = L.lamS[3 * me + q], lset = L.lamSet[3 * me + q], dv = ls - c.l[q];
          L.gS[3 * me + q] = c.e[q];
          dpart += dv * dv;
          bpart += L.rec[(PGS_RC + q) * PGS_SMAX + me] * fmax(fabs(ls - lset), fabs(c.l[q] - lset));
          npart += ls * ls;
        }
        L.stS[me] = (unsigned char)c.st;
      }
      for (int o = 32; o > 0; o >>= 1) {
        dpart += __shfl_xor(dpart, o, 64);
        bpart += __shfl_xor(bpart, o, 64);
        npart += __shfl_xor(npart, o, 64);
      }
      if (ln == 0) {
        red[3 * wu] = dpart;
        red[3 * wu + 1] = bpart;
        red[3 * wu + 2] = npart;
      }
    }
    prog += nsp;
    ++nsweep;
    __syncthreads();
    if (prog > (1 << 30)) {   // the count of solved contacts starts over
      prog = 0;
      __syncthreads();
      if (tid == 0) L.cprog = 0;
      __syncthreads();
    }
    double dsum = 0.0, B = 0.0, nsum = 0.0;   // every thread takes the same sums
    for (int w = 0; 64 * w < nS; ++w) {
      dsum += red[3 * w];
      B += red[3 * w + 1];
      nsum += red[3 * w + 2];
    }
    const double diff = sqrt(dsum), nl = sqrt(nsum);
    eps = nl > 0.0 ? diff / nl : (diff == 0.0 ? 0.0 : INFINITY);
    const bool perr = L.perr != 0;
    if (perr) eps = NAN;   // the ring sweep lost its count: stop and report eps = NaN
    const bool stop = eps <= tol || perr;
    B *= 1.0 + 1e-12;
    // ---- verify the skipped contacts (all settled at once when B < Rmin)
    bool grow = false;
    if (L.zflag != 0 || !(B < L.Rmin)) {
      if (tid == 0) {
        L.nu = 0;
        L.flag = 0;
      }
      __syncthreads();
      for (int c = tid; c < nc; c += PGS_NT) {
        if (L.inS[c]) continue;
        const double g = gnSet[c], rb = swn[c] * B;
        if (!(g - rb > 1e-13 * (fabs(g) + rb))) L.ulist[atomicAdd(&L.nu, 1)] = (unsigned short)c;
      }
      __syncthreads();
      int nu = L.nu;
      nexact += nu;
      const bool rebase = nexact >= nc - nS;
      if (rebase) {   // all of them
        nexact = 0;
        __syncthreads();
        if (tid == 0) L.nu = 0;
        __syncthreads();
        for (int c = tid; c < nc; c += PGS_NT)
          if (!L.inS[c]) L.ulist[atomicAdd(&L.nu, 1)] = (unsigned short)c;
        __syncthreads();
        nu = L.nu;
      }
      // exact gaps at the contacts' turn (at) and at the sweep's end (ae), four
      // contacts at a time, their rows of W in flight together
      for (int u = 4 * wv; u < nu; u += 4 * PGS_NW) {
        int c[4];
        double at[4] = {0.0, 0.0, 0.0, 0.0}, ae[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4; ++k) c[k] = L.ulist[min(u + k, nu - 1)];
        for (int q = ln; q < ldS; q += 64) {
          const int s = L.Sidx[q / 3];
          const double set = L.lamSet[q], de = L.lamS[q] - set, d0 = L.lamS0[q] - set;
          const long col = 3L * s + q % 3;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const double w = h2 * (double)W[(3L * c[k]) * m + col];
            at[k] = fma(w, s < c[k] ? de : d0, at[k]);
            ae[k] = fma(w, de, ae[k]);
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          for (int o = 32; o > 0; o >>= 1) {
            at[k] += __shfl_xor(at[k], o, 64);
            ae[k] += __shfl_xor(ae[k], o, 64);
          }
          if (ln == 0 && u + k < nu) {
            const double g = gnSet[c[k]];
            if (g + at[k] < 0.0) {
              L.inS[c[k]] = 1;
              L.flag = 1;
            }
            if (rebase) gnSet[c[k]] = g + ae[k];
          }
        }
      }
      __syncthreads();
      grow = L.flag != 0 && !perr;
      if (rebase && !grow) {
        for (int r = tid; r < ldS; r += PGS_NT) L.lamSet[r] = L.lamS[r];
        built = true;   // a new settle threshold
        __threadfence_block();
        __syncthreads();
      }
    }
    if (grow) {
      // a skipped contact was not a no-op: restart the sweep with a larger S
      for (int r = tid; r < ldS; r += PGS_NT) lam[3 * L.Sidx[r / 3] + r % 3] = L.lamS0[r];
      need_build = true;
      __threadfence_block();
      __syncthreads();
      continue;
    }
    ++sweep;
    if (stop) break;
  }
  for (int r = tid; r < ldS; r += PGS_NT) lam[3 * L.Sidx[r / 3] + r % 3] = L.lamS[r];
  for (int i = tid; i < nS; i += PGS_NT) status[L.Sidx[i]] = (int8_t)L.stS[i];
  if (tid == 0) {
    *sweeps_out = sweep;
    *eps_out = eps;
  }
}

template <class TW>
__global__ __launch_bounds__(PGS_NT) void k_pgs_active(int nc, const TW *__restrict__ W,
                                                       const double *__restrict__ d, const double *__restrict__ g0,
                                                       const double *__restrict__ mu, double h2,
                                                       double *__restrict__ lam, int8_t *__restrict__ status,
                                                       int max_sweeps, double tol, int j_inner,
                                                       int *__restrict__ sweeps_out, double *__restrict__ eps_out,
                                                       double *__restrict__ Wss, double *__restrict__ gnSet,
                                                       const double *__restrict__ swn, int *__restrict__ ctl,
                                                       const int *__restrict__ preSidx, const int *__restrict__ preN,
                                                       const double *__restrict__ preRec,
                                                       const double *__restrict__ preGS) {
  extern __shared__ double lds_raw[];
  PgsLds &L = *reinterpret_cast<PgsLds *>(lds_raw);
  pgs_active_body<TW>(L, nc, W, d, g0, mu, h2, lam, status, max_sweeps, tol, j_inner, sweeps_out, eps_out, Wss,
                      gnSet, swn, ctl, preSidx, *preN, preRec, preGS);
}

// y[i] = x0[i] + h2 sum over the contacts c with a non-zero block of v
// (ascending) of M[(3c + a) m + i] v[3c + a], by one workgroup (M symmetric,
// rows of M read for its columns).  The order of every sum is that of
// k_sym_gemv_sparse (one 64-row block at a time, wave w takes list entries
// w, w + 8, ..., the eight partial sums added in wave order), so the result
// is bit-for-bit the per-scene kernel's.  The contacts taken are those with
// a non-zero block of nzv (the forces lambda, also when v is f = C^T lambda,
// as there); list (LDS) receives them, part (LDS) holds 8 x 64 partial sums.
template <class TM>
__device__ void wg_sym_gemv_sparse(int nc, const TM *__restrict__ M, const double *__restrict__ x0,
                                   const double *__restrict__ v, const double *__restrict__ nzv, double h2,
                                   double *__restrict__ y, unsigned short *list, int *count, double *part) {
  static_assert(PGS_NT == SG_NT, "the per-scene kernel's wave count");
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const long m = 3L * nc;
  if (wv == 0) {
    int cnt = 0;
    for (int c0 = 0; c0 < nc; c0 += 64) {
      const int c = c0 + ln;
      const bool nz = c < nc && block_nonzero(nzv, c);
      const unsigned long long bal = __ballot(nz);
      if (nz) list[cnt + __popcll(bal & ((1ull << ln) - 1ull))] = (unsigned short)c;
      cnt += __popcll(bal);
    }
    if (ln == 0) *count = cnt;
  }
  __syncthreads();
  const int n = *count;
  for (long i0 = 0; i0 < m; i0 += 64) {
    const long i = i0 + ln;
    double s = 0.0;
    if (i < m) {
#pragma unroll 4
      for (int q = wv; q < n; q += SG_NW) {
        const long r = 3L * list[q];
        s = fma((double)M[r * m + i], v[r], s);
        s = fma((double)M[(r + 1) * m + i], v[r + 1], s);
        s = fma((double)M[(r + 2) * m + i], v[r + 2], s);
      }
    }
    part[wv * 64 + ln] = s;
    __syncthreads();
    if (wv == 0 && i < m) {
      double t = 0.0;
      for (int w = 0; w < SG_NW; ++w) t += part[w * 64 + ln];
      y[i] = x0[i] + h2 * t;
    }
    __syncthreads();
  }
}

// ---- batched Newton loops --------------------------------------------------
//
// Algorithm 3's Newton loops (steps 1-4) of a group of scenes, one launch per
// step for all of them (blockIdx.y: the scene; the iterations that only scenes
// of few contacts have are one launch, k_batch_small): frames and gaps at the last
// proximity (the warm start in the new frames), W_k = C_k W_H C_k^T, the PGS
// start gaps g0 = d + W~ lambda and the set, the active-set PGS (one workgroup
// per scene), and the world forces f = C^T lambda with the proximity p = p_free
// + h^2 W_H f (Eq. 31).  The bodies are those of the per-scene kernels, so a
// step's results do not depend on the path it took.  One workgroup for a
// scene's whole loop streamed W_H and W through a single compute unit, a third
// of the loop's time: groups of three scenes of 10 to 500 contacts took 12.7 ms
// a loop of five iterations, and take 9.6 ms, of which the PGS has 9.2.  The
// iterations of a group run in step, so each waits for its largest set; that is
// the same scene in most of them.
// The task table as the device reads it: the same layout with every pointer
// in the global address space, so that the code inlined below uses global
// loads and their counters (a pointer read from memory is otherwise generic).
template <class T>
using gptr = __attribute__((address_space(1))) T *;
struct NewtonTaskG {
  int nc, n_newton, max_sweeps, j_inner;
  double tol, h;
  gptr<const StepCtx> ctx;
  gptr<const double> WH, pfree, pstart, mu;
  gptr<double> W, p, f, C, dk, lam, eps;
  gptr<double> g, Wss, gnSet, swn, rec, gS;
  gptr<int8_t> status;
  gptr<int> sweeps, ctl, Sidx, nS;
};
static_assert(sizeof(NewtonTaskG) == sizeof(NewtonTask) && offsetof(NewtonTaskG, nS) == offsetof(NewtonTask, nS),
              "device view of the task table");

// Scene blockIdx.y of the launch.
__device__ __forceinline__ const NewtonTaskG &newton_task(const NewtonTask *__restrict__ tasks,
                                                          const NewtonBatchIdx &ids) {
  return reinterpret_cast<const NewtonTaskG *>(tasks)[ids.idx[blockIdx.y]];
}
__global__ void k_batch_directions(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids, int k) {
  const NewtonTaskG &t = newton_task(tasks, ids);
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= t.n_newton || c >= t.nc) return;
  const gptr<const double> p = k == 0 ? t.pfree : (gptr<const double>)t.p;
  directions_contact(c, (const StepCtx *)t.ctx, (const double *)p, (const double *)t.pfree, (const double *)t.pstart, (const double *)t.f, (double *)t.C,
                     (double *)t.dk, (double *)t.lam, 0, nullptr);
}
__global__ void k_batch_update_W(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids, int k) {
  const NewtonTaskG &t = newton_task(tasks, ids);
  const long blk = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= t.n_newton || blk >= (long)t.nc * t.nc) return;
  update_W_block(t.nc, (const double *)t.WH, (const double *)t.C, (double *)t.W, blk);
}
__global__ __launch_bounds__(SG_NT) void k_batch_gaps(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids, int k) {
  const NewtonTaskG &t = newton_task(tasks, ids);
  if (k >= t.n_newton || 64 * (int)blockIdx.x >= 3 * t.nc) return;
  sym_gemv_sparse<double>(t.nc, (const double *)t.W, (const double *)t.dk, (const double *)t.lam, t.h * t.h,
                          (double *)t.g, nullptr, nullptr, nullptr);
}
__global__ __launch_bounds__(SG_NT) void k_batch_proximity(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids,
                                                           int k) {
  const NewtonTaskG &t = newton_task(tasks, ids);
  if (k >= t.n_newton || 64 * (int)blockIdx.x >= 3 * t.nc) return;
  sym_gemv_sparse<double>(t.nc, (const double *)t.WH, (const double *)t.pfree, (const double *)t.lam, t.h * t.h,
                          (double *)t.p, (const double *)t.C, (const double *)t.lam, (double *)t.f);
}
__global__ __launch_bounds__(256) void k_batch_gather(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids, int k) {
  const NewtonTaskG &t = newton_task(tasks, ids);
  if (k >= t.n_newton) return;
  pgs_gather<double>(t.nc, (const double *)t.W, (const double *)t.g, (const double *)t.lam, (const double *)t.mu,
                     t.h * t.h, (int *)t.Sidx, (int *)t.nS, (double *)t.gnSet, (double *)t.swn,
                     (double *)t.Wss, (double *)t.rec, (double *)t.gS);
}
__global__ __launch_bounds__(PGS_NT) void k_batch_pgs(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids, int k) {
  extern __shared__ double lds_raw[];
  PgsLds &L = *reinterpret_cast<PgsLds *>(lds_raw);
  const NewtonTaskG &t = newton_task(tasks, ids);
  if (k >= t.n_newton) return;
  pgs_active_body<double>(L, t.nc, (const double *)t.W, (const double *)t.dk, (const double *)t.g,
                          (const double *)t.mu, t.h * t.h, (double *)t.lam, (int8_t *)t.status, t.max_sweeps,
                          t.tol, t.j_inner, (int *)t.sweeps + k, (double *)t.eps + k, (double *)t.Wss,
                          (double *)t.gnSet, (const double *)t.swn, (int *)t.ctl, (const int *)t.Sidx, *(const int *)t.nS,
                          (const double *)t.rec, (const double *)t.gS);
}

// The iterations from k0 on of scenes of few contacts, in one launch: a
// workgroup runs its scene's whole loop, one step after the other.
__global__ __launch_bounds__(PGS_NT) void k_batch_small(const NewtonTask *__restrict__ tasks, NewtonBatchIdx ids,
                                                        int k0) {
  extern __shared__ double lds_raw[];
  PgsLds &L = *reinterpret_cast<PgsLds *>(lds_raw);
  const NewtonTaskG &tg = newton_task(tasks, ids);
  struct {
    int nc, n_newton, max_sweeps, j_inner;
    double tol, h;
    const StepCtx *ctx;
    const double *WH, *pfree, *pstart, *mu;
    double *W, *p, *f, *C, *dk, *lam, *eps;
    double *g, *Wss, *gnSet, *swn;
    int8_t *status;
    int *sweeps, *ctl;
  } t{tg.nc, tg.n_newton, tg.max_sweeps, tg.j_inner, tg.tol, tg.h, (const StepCtx *)tg.ctx,
      (const double *)tg.WH, (const double *)tg.pfree, (const double *)tg.pstart, (const double *)tg.mu,
      (double *)tg.W, (double *)tg.p, (double *)tg.f, (double *)tg.C, (double *)tg.dk, (double *)tg.lam,
      (double *)tg.eps, (double *)tg.g, (double *)tg.Wss, (double *)tg.gnSet, (double *)tg.swn,
      (int8_t *)tg.status, (int *)tg.sweeps, (int *)tg.ctl};
  const int nc = t.nc, tid = threadIdx.x;
  const long m = 3L * nc;
  const double h2 = t.h * t.h;
  for (int k = k0; k < t.n_newton; ++k) {
    for (int c = tid; c < nc; c += PGS_NT)
      directions_contact(c, t.ctx, k == 0 ? t.pfree : t.p, t.pfree, t.pstart, t.f, t.C, t.dk, t.lam, 0, nullptr);
    __syncthreads();
    for (long blk = tid; blk < (long)nc * nc; blk += PGS_NT) update_W_block(nc, t.WH, t.C, t.W, blk);
    __syncthreads();
    wg_sym_gemv_sparse<double>(nc, t.W, t.dk, t.lam, t.lam, h2, t.g, L.ulist, &L.nu, L.lamS);
    for (int c = tid; c < nc; c += PGS_NT) {
      t.gnSet[c] = t.g[3 * c];
      t.swn[c] = sqrt(h2 * t.W[(3L * c) * m + 3L * c]);
    }
    __syncthreads();
    // no prepared set: the body builds it
    pgs_active_body<double>(L, nc, t.W, t.dk, t.g, t.mu, h2, t.lam, t.status, t.max_sweeps, t.tol, t.j_inner,
                            t.sweeps + k, t.eps + k, t.Wss, t.gnSet, t.swn, t.ctl, nullptr, PGS_WAVE_MAX + 1,
                            nullptr, nullptr);
    __syncthreads();
    for (long e = tid; e < m; e += PGS_NT) t.f[e] = world_force(t.C, t.lam, e / 3, (int)(e % 3));
    __syncthreads();
    wg_sym_gemv_sparse<double>(nc, t.WH, t.pfree, t.f, t.lam, h2, t.p, L.ulist, &L.nu, L.lamS);
  }
}

// ---- directions updated before every local solve, on the register chain ----
//
// The per-constraint Gauss-Seidel (R18, k_pgs_pc) with the structure of
// k_pgs_active: only contacts with a force or a negative normal gap can
// change (a contact with no force whose gap at its turn is >= 0 stays
// separated: a no-op), so the sweep runs over the set S of those contacts
// alone.  Wave 0 holds their proximities P (world frame) in registers; at
// contact a's turn it takes its frame and gap at P_a, the block
// W~_aa = h^2 C_a W_H,aa C_a^T, the gap without the own force, the local
// solve and f_a = C_a^T lambda_a with the same arithmetic as k_pgs_pc, then
// every lane adds h^2 W_H(own rows, a) (f_a - f_a^old) to its proximities.
// After a sweep every contact c outside S is verified to have been a no-op:
// its proximity at its turn is P_c^set + h^2 sum_{b in S} W_H,cb
// (f_b^turn - f_b^set) (forces of S contacts before c in this sweep, after
// it from the previous sweep); the signed distance is 1-Lipschitz and
// |h^2 W_H,cb| <= h sqrt(tr W_H,cc) h sqrt(tr W_H,bb) for the PSD W_H, so
// phi_set(c) > h sqrt(tr W_H,cc) B with
// B = sum_b h sqrt(tr W_H,bb) max(|f_b^new - f_b^set|, |f_b^old - f_b^set|)
// settles c, and the others get their exact proximity and gap.  A violation
// adds the contact to S and restarts the sweep from its start state; a set
// beyond 128 contacts hands over to k_pgs_pc (ctl[0] = 1, the sweep in
// ctl[1], the proximity of the hand-over state in Pset).
constexpr int PCA_MAX = 128;   // contacts of S in the single-wave chain
constexpr int PCA_RW = 26;     // record of a contact of S, see PcaLds
struct PcaLds {
  double P[3 * PCA_MAX];       // proximity of S (the chain's registers between sweeps)
  // per contact of S: 0-5 W_H,aa (w00 w01 w02 w11 w12 w22), 6 mu, 7-9 p_start,
  // 10-12 lambda, 13-21 frame rows, 22-24 world force f, 25 unused
  double rec[PCA_MAX * PCA_RW];
  double f0[3 * PCA_MAX];      // forces of S at the sweep's start
  double fset[3 * PCA_MAX];    // ... at the set's start state
  double part[8 * 64];         // partial sums of the proximity product
  double red[48];
  int Sidx[PCA_MAX];
  unsigned char stS[PCA_MAX];
  int wcount[64];
  unsigned short ulist[PGS_MAX_NC];
  unsigned char inS[PGS_MAX_NC];
  int nS, flag, stop, nu;
  int cprog, perr;   // two-wave sweep: contacts done by the solving wave; a wait ran out
};
static_assert(sizeof(PcaLds) <= 160 * 1024, "per-constraint chain state must fit one CU's LDS");

struct PcaRec {
  double2 r2[PCA_RW / 2];
  __device__ double operator[](int q) const { return (q & 1) ? r2[q >> 1].y : r2[q >> 1].x; }
};
__device__ inline void pca_rec(PcaRec &c, const PcaLds &L, int i) {
  const double2 *rp = reinterpret_cast<const double2 *>(L.rec + PCA_RW * i);
#pragma unroll
  for (int q = 0; q < PCA_RW / 2; ++q) c.r2[q] = rp[q];
}

// contact_frame with each normalisation by the refined reciprocal square
// root of the squared length (the length itself is that square times it):
// within an ulp or two of the square roots and divisions, and a short
// dependent chain; the frame of every visit of the chain.
__device__ inline void contact_frame_rcp(const icr_obstacle &obs, double t0, double t1, const double pc[3],
                                         const double ps[3], double F[3][3], double delta[3]) {
  double n[3], phi;
  {
#pragma clang fp contract(off)
    const double c[3] = {obs.c0[0] + obs.vel[0] * t1, obs.c0[1] + obs.vel[1] * t1, obs.c0[2] + obs.vel[2] * t1};
    const double r0 = pc[0] - c[0], r1 = pc[1] - c[1], r2 = pc[2] - c[2];
    if (obs.kind == 1) {
      const double d2 = r0 * r0 + r1 * r1 + r2 * r2;
      const double id = frsqrt(d2);
      n[0] = r0 * id;
      n[1] = r1 * id;
      n[2] = r2 * id;
      phi = d2 * id - obs.radius;
    } else {
      n[0] = obs.normal[0];
      n[1] = obs.normal[1];
      n[2] = obs.normal[2];
      phi = r0 * obs.normal[0] + r1 * obs.normal[1] + r2 * obs.normal[2];
    }
  }
  int ax = 0;
  double am = fabs(n[0]);
  if (fabs(n[1]) < am) {
    ax = 1;
    am = fabs(n[1]);
  }
  if (fabs(n[2]) < am) ax = 2;
  const double en = n[ax];
  double ta[3] = {-en * n[0], -en * n[1], -en * n[2]};
  ta[ax] += 1.0;
  const double itn = frsqrt(ta[0] * ta[0] + ta[1] * ta[1] + ta[2] * ta[2]);
  ta[0] *= itn;
  ta[1] *= itn;
  ta[2] *= itn;
  const double tb[3] = {n[1] * ta[2] - n[2] * ta[1], n[2] * ta[0] - n[0] * ta[2], n[0] * ta[1] - n[1] * ta[0]};
  double rel[3];
  for (int a = 0; a < 3; ++a) {
    const double uo = (obs.c0[a] + obs.vel[a] * t1) - (obs.c0[a] + obs.vel[a] * t0);
    rel[a] = pc[a] - ps[a] - uo;
  }
  for (int a = 0; a < 3; ++a) {
    F[0][a] = n[a];
    F[1][a] = ta[a];
    F[2][a] = tb[a];
  }
  delta[0] = phi;
  delta[1] = ta[0] * rel[0] + ta[1] * rel[1] + ta[2] * rel[2];
  delta[2] = tb[0] * rel[0] + tb[1] * rel[1] + tb[2] * rel[2];
}

// One visit of the chain: contact i, its proximity in lane i % 64.
template <int J>
__device__ inline void pca_step(int i, const BlkCol &X, const PcaRec &c, double (&g)[3], PcaLds &L, int j_inner,
                                int ln, const icr_obstacle &obs, double t0, double t1, double h2) {
  const int li = i & 63;
  const double pa[3] = {readlane_f64(g[0], li), readlane_f64(g[1], li), readlane_f64(g[2], li)};
  const double ps[3] = {c[7], c[8], c[9]};
  double F[3][3], delta[3];
  contact_frame_rcp(obs, t0, t1, pa, ps, F, delta);
  const double wh[3][3] = {{c[0], c[1], c[2]}, {c[1], c[3], c[4]}, {c[2], c[4], c[5]}};
  double B[3][3];   // W_H,aa C_a^T
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) B[a][b] = wh[a][0] * F[b][0] + wh[a][1] * F[b][1] + wh[a][2] * F[b][2];
  double w[3][3];
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) w[a][b] = h2 * (F[a][0] * B[0][b] + F[a][1] * B[1][b] + F[a][2] * B[2][b]);
  for (int a = 0; a < 3; ++a)   // exactly symmetric block
    for (int b = 0; b < a; ++b) w[b][a] = w[a][b];
  const double fo[3] = {c[22], c[23], c[24]};
  double lr[3], dd[3];
  for (int a = 0; a < 3; ++a) lr[a] = F[a][0] * fo[0] + F[a][1] * fo[1] + F[a][2] * fo[2];
  for (int a = 0; a < 3; ++a) dd[a] = delta[a] - (w[a][0] * lr[0] + w[a][1] * lr[1] + w[a][2] * lr[2]);
  const PgsRec rc = make_record<true>(w, c[6]);
  const Local r = local_solve_rec<J>(rc, dd, j_inner);
  double fn[3], df[3];
  for (int q = 0; q < 3; ++q) {
    fn[q] = F[0][q] * r.l[0] + F[1][q] * r.l[1] + F[2][q] * r.l[2];
    df[q] = fn[q] - fo[q];
  }
  if (ln == 0) {
    double *lp = L.rec + PCA_RW * i;
    for (int q = 0; q < 3; ++q) {
      lp[10 + q] = r.l[q];
      lp[22 + q] = fn[q];
      for (int k = 0; k < 3; ++k) lp[13 + 3 * q + k] = F[q][k];
    }
    L.stS[i] = (unsigned char)r.st;
  }
  blk_apply(g, X, df[0], df[1], df[2]);
}

// Column i's blocks of the rows of wave w (h^2 W_H,SS padded to nsp contacts).
__device__ __forceinline__ void pca_load(BlkCol &X, const BlkBuf &B, int i, int nsp, int w, int ln) {
  blk_load(X, B, 8u * (unsigned)(i * (nsp * PGS_BLK) + BLK_GROUP * w), ln);
}

template <int J>
__device__ __forceinline__ void pca_chain(int nS, const BlkBuf &Wb, PcaLds &L, int j_inner,
                                          const icr_obstacle &obs, double t0, double t1, double h2) {
  const int ln = threadIdx.x & 63;
  double g[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) g[q] = ln < nS ? L.P[3 * ln + q] : 0.0;
  const int last = nS - 1;
  BlkCol A, B;
  PcaRec rA, rB;
  pca_load(A, Wb, 0, 64, 0, ln);
  pca_load(B, Wb, min(1, last), 64, 0, ln);
  pca_rec(rA, L, 0);
  for (int i = 0; i < nS; i += 2) {
    pca_rec(rB, L, min(i + 1, last));
    pca_step<J>(i, A, rA, g, L, j_inner, ln, obs, t0, t1, h2);
    pca_load(A, Wb, min(i + 2, last), 64, 0, ln);
    if (i + 1 < nS) {
      pca_rec(rA, L, min(i + 2, last));
      pca_step<J>(i + 1, B, rB, g, L, j_inner, ln, obs, t0, t1, h2);
    }
    pca_load(B, Wb, min(i + 3, last), 64, 0, ln);
  }
  if (ln < nS) {
#pragma unroll
    for (int q = 0; q < 3; ++q) L.P[3 * ln + q] = g[q];
  }
}

// A set of 65..128 contacts is swept by two waves as in chain_sweep: wave w
// keeps the proximities of contacts 64 w .. 64 w + 63, solves those
// contacts while the other wave adds each published force change to its own
// proximities, then applies the other half's changes.  The applying wave
// takes the change as the published world force minus the force at the
// sweep's start, so every proximity receives the same products in the same
// order as in the one-wave sweep.
template <int J>
__device__ inline void pca_pair_solve(int b, int e, const BlkBuf &Wb, PcaLds &L, int j_inner, int ln,
                                      int w, double (&g)[3], const icr_obstacle &obs, double t0, double t1,
                                      double h2) {
  if (b >= e) return;
  const int last = e - 1;
  BlkCol A, B;
  PcaRec rA, rB;
  pca_load(A, Wb, b, 128, w, ln);
  pca_load(B, Wb, min(b + 1, last), 128, w, ln);
  pca_rec(rA, L, b);
  for (int i = b; i < e; i += 2) {
    pca_rec(rB, L, min(i + 1, last));
    pca_step<J>(i, A, rA, g, L, j_inner, ln, obs, t0, t1, h2);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (ln == 0) __hip_atomic_store(&L.cprog, i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    pca_load(A, Wb, min(i + 2, last), 128, w, ln);
    if (i + 1 < e) {
      pca_rec(rA, L, min(i + 2, last));
      pca_step<J>(i + 1, B, rB, g, L, j_inner, ln, obs, t0, t1, h2);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (ln == 0) __hip_atomic_store(&L.cprog, i + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    pca_load(B, Wb, min(i + 3, last), 128, w, ln);
  }
}
__device__ inline void pca_pair_apply_one(int i, const BlkCol &X, PcaLds &L, double (&g)[3]) {
  for (int spin = 0; __hip_atomic_load(&L.cprog, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= i; ++spin) {
    if (spin == RING_SPIN) {
      __hip_atomic_store(&L.perr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      break;
    }
    if ((spin & 255) == 255 && __hip_atomic_load(&L.perr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0)
      break;
    __builtin_amdgcn_s_sleep(1);
  }
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  const double *rp = L.rec + PCA_RW * i + 22;
  const double d0 = rp[0] - L.f0[3 * i], d1 = rp[1] - L.f0[3 * i + 1], d2 = rp[2] - L.f0[3 * i + 2];
  blk_apply(g, X, d0, d1, d2);
}
__device__ inline void pca_pair_apply(int b, int e, const BlkBuf &Wb, PcaLds &L, int ln, int w,
                                      double (&g)[3]) {
  if (b >= e) return;
  const int last = e - 1;
  BlkCol A, B;
  pca_load(A, Wb, b, 128, w, ln);
  pca_load(B, Wb, min(b + 1, last), 128, w, ln);
  for (int i = b; i < e; i += 2) {
    pca_pair_apply_one(i, A, L, g);
    pca_load(A, Wb, min(i + 2, last), 128, w, ln);
    if (i + 1 < e) pca_pair_apply_one(i + 1, B, L, g);
    pca_load(B, Wb, min(i + 3, last), 128, w, ln);
  }
}
template <int J>
__device__ __forceinline__ void pca_pair(int nS, const BlkBuf &Wb, PcaLds &L, int j_inner,
                                         const icr_obstacle &obs, double t0, double t1, double h2, int w) {
  const int ln = threadIdx.x & 63, c = 64 * w + ln, h = min(64, nS);
  double g[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) g[q] = c < nS ? L.P[3 * c + q] : 0.0;
  if (w == 0) {
    pca_pair_solve<J>(0, h, Wb, L, j_inner, ln, w, g, obs, t0, t1, h2);
    pca_pair_apply(h, nS, Wb, L, ln, w, g);
  } else {
    pca_pair_apply(0, h, Wb, L, ln, w, g);
    pca_pair_solve<J>(h, nS, Wb, L, j_inner, ln, w, g, obs, t0, t1, h2);
  }
  if (c < nS) {
#pragma unroll
    for (int q = 0; q < 3; ++q) L.P[3 * c + q] = g[q];
  }
}

// Exact proximity of a contact c outside S at its turn in the last sweep,
// by one wave (all lanes return it): Pset_c + h^2 sum_{b in S} W_H,cb
// (f_b^turn - f_b^set).
__device__ inline void pca_turn_proximity(int c, int nS, int m, const double *__restrict__ WH,
                                          const double *__restrict__ Pset, double h2, const PcaLds &L, int ln,
                                          double pt[3]) {
  double a[3] = {0.0, 0.0, 0.0};
  for (int q = ln; q < 3 * nS; q += 64) {
    const int b = L.Sidx[q / 3];
    const double fnew = L.rec[PCA_RW * (q / 3) + 22 + q % 3];
    const double d = ((b < c) ? fnew : L.f0[q]) - L.fset[q];
#pragma unroll
    for (int r = 0; r < 3; ++r) a[r] = fma(h2 * WH[(3L * c + r) * m + 3L * b + q % 3], d, a[r]);
  }
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    for (int o = 32; o > 0; o >>= 1) a[r] += __shfl_xor(a[r], o, 64);
    pt[r] = Pset[3 * c + r] + a[r];
  }
}

__global__ __launch_bounds__(PGS_NT) void k_pgs_pca(int nc, const StepCtx *__restrict__ ctx,
                                                    const double *__restrict__ WH, const double *__restrict__ pfree,
                                                    const double *__restrict__ pin, const double *__restrict__ pstart,
                                                    const double *__restrict__ mu, double h2, double *__restrict__ f,
                                                    double *__restrict__ C, double *__restrict__ lam,
                                                    int8_t *__restrict__ status, int max_sweeps, double tol,
                                                    int j_inner, int *__restrict__ sweeps_out,
                                                    double *__restrict__ eps_out, double *__restrict__ Wss,
                                                    double *__restrict__ Pset, double *__restrict__ gnSet,
                                                    double *__restrict__ swn, int *__restrict__ ctl) {
  extern __shared__ double lds_raw[];
  PcaLds &L = *reinterpret_cast<PcaLds *>(lds_raw);
  const int m = 3 * nc;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const icr_obstacle obs = ctx->obs;
  const double t0 = ctx->t0, t1 = ctx->t0 + ctx->h;
  for (int c = tid; c < nc; c += PGS_NT) {
    const long d = 3L * c;
    swn[c] = sqrt(h2 * (WH[d * m + d] + WH[(d + 1) * m + d + 1] + WH[(d + 2) * m + d + 2]));
    L.inS[c] = 0;
  }
  for (int e = tid; e < m; e += PGS_NT) Pset[e] = pin[e];
  if (tid == 0) {
    ctl[0] = 0;
    ctl[1] = 0;
    L.stop = 0;
    L.perr = 0;
  }
  __syncthreads();
  int sweep = 0, nS = 0, nsp = 64;
  double eps = 0.0;
  bool need_build = true, first = true;
  while (sweep < max_sweeps) {
    if (need_build) {
      // proximity of the set's start state (given for the first set)
      if (!first) wg_sym_gemv_sparse<double>(nc, WH, pfree, f, f, h2, Pset, L.ulist, &L.nu, L.part);
      // normal gaps there; members: a force, a negative gap, or an earlier violation
      for (int c = tid; c < nc; c += PGS_NT) {
        const double pc[3] = {Pset[3 * c], Pset[3 * c + 1], Pset[3 * c + 2]};
        const double ps[3] = {pstart[3 * c], pstart[3 * c + 1], pstart[3 * c + 2]};
        double F[3][3], delta[3];
        contact_frame(obs, t0, t1, pc, ps, F, delta);
        gnSet[c] = delta[0];
        const bool nz = f[3 * c] != 0.0 || f[3 * c + 1] != 0.0 || f[3 * c + 2] != 0.0;
        if (nz || delta[0] < 0.0) L.inS[c] = 1;
      }
      __syncthreads();
      const int nwin = (nc + 63) / 64;
      for (int w = wv; w < nwin; w += PGS_NW) {
        const int c = 64 * w + ln;
        const unsigned long long bal = __ballot(c < nc && L.inS[c]);
        if (ln == 0) L.wcount[w] = __popcll(bal);
      }
      __syncthreads();
      if (tid == 0) {
        int acc = 0;
        for (int w = 0; w < nwin; ++w) {
          const int t = L.wcount[w];
          L.wcount[w] = acc;
          acc += t;
        }
        L.nS = acc;
      }
      __syncthreads();
      nS = __builtin_amdgcn_readfirstlane(L.nS);
      if (nS > PCA_MAX) {   // hand over: f and Pset hold the sweep-start state
        if (tid == 0) {
          ctl[0] = 1;
          ctl[1] = sweep;
        }
        return;
      }
      for (int w = wv; w < nwin; w += PGS_NW) {
        const int c = 64 * w + ln;
        const bool in = c < nc && L.inS[c];
        const unsigned long long bal = __ballot(in);
        if (in) L.Sidx[L.wcount[w] + __popcll(bal & ((1ull << ln) - 1ull))] = c;
      }
      __syncthreads();
      nsp = pgs_wave_pad(nS);
      for (int i = tid; i < nS; i += PGS_NT) {
        const long d = 3L * L.Sidx[i];
        double *rc = L.rec + PCA_RW * i;
        rc[0] = WH[d * m + d];
        rc[1] = WH[d * m + d + 1];
        rc[2] = WH[d * m + d + 2];
        rc[3] = WH[(d + 1) * m + d + 1];
        rc[4] = WH[(d + 1) * m + d + 2];
        rc[5] = WH[(d + 2) * m + d + 2];
        rc[6] = mu[L.Sidx[i]];
        for (int q = 0; q < 3; ++q) {
          rc[7 + q] = pstart[d + q];
          rc[22 + q] = f[d + q];
        }
      }
      for (int r = tid; r < 3 * nS; r += PGS_NT) {
        const long e = 3L * L.Sidx[r / 3] + r % 3;
        L.P[r] = Pset[e];
        L.fset[r] = f[e];
      }
      // h^2 W_H,SS blocked [i][c] (rows of contact c, columns of contact i),
      // diagonal blocks included
      const long nel = (long)nS * nsp * PGS_BLK;
      for (long e = tid; e < nel; e += PGS_NT) {
        const int per = nsp * PGS_BLK, i = (int)(e / per), r = (int)(e % per);
        int l, j;
        blk_index(r % BLK_GROUP, l, j);
        const int cc = 64 * (r / BLK_GROUP) + l;
        double v = 0.0;
        if (cc < nS) v = h2 * WH[(3L * L.Sidx[i] + j % 3) * m + 3L * L.Sidx[cc] + j / 3];
        Wss[e] = v;
      }
      __threadfence_block();
      __syncthreads();
      need_build = false;
      first = false;
    }
    // ---- one sweep over S from its start state
    for (int r = tid; r < 3 * nS; r += PGS_NT) L.f0[r] = L.rec[PCA_RW * (r / 3) + 22 + r % 3];
    if (tid == 0) {
      L.flag = 0;
      L.nu = 0;
      L.cprog = 0;
    }
    __syncthreads();
    if (nS > 0) {
      const BlkBuf buf(Wss, 8u * PGS_BLK * (unsigned)nsp * (unsigned)nS);
      const int wu = __builtin_amdgcn_readfirstlane(wv);
      if (nsp == 64) {
        if (wv == 0) {
          if (j_inner == 8)
            pca_chain<8>(nS, buf, L, j_inner, obs, t0, t1, h2);
          else
            pca_chain<0>(nS, buf, L, j_inner, obs, t0, t1, h2);
        }
      } else if (wv < 2) {
        if (j_inner == 8)
          pca_pair<8>(nS, buf, L, j_inner, obs, t0, t1, h2, wu);
        else
          pca_pair<0>(nS, buf, L, j_inner, obs, t0, t1, h2, wu);
      }
    }
    __syncthreads();
    // eps = |f_i - f_{i-1}| / |f_i| (forces outside S stay zero), and B
    double dpart = 0.0, bpart = 0.0, npart = 0.0;
    for (int i = tid; i < nS; i += PGS_NT) {
      const double *rc = L.rec + PCA_RW * i;
      double dnew = 0.0, dold = 0.0;
      for (int q = 0; q < 3; ++q) {
        const double fn = rc[22 + q], fo = L.f0[3 * i + q], fs = L.fset[3 * i + q];
        dpart += (fn - fo) * (fn - fo);
        npart += fn * fn;
        dnew += (fn - fs) * (fn - fs);
        dold += (fo - fs) * (fo - fs);
      }
      bpart += sqrt(h2 * (rc[0] + rc[3] + rc[5])) * sqrt(fmax(dnew, dold));
    }
    block_sum3(dpart, bpart, npart, L.red);
    if (tid == 0) {
      const double diff = sqrt(dpart), nf = sqrt(npart);
      eps = nf > 0.0 ? diff / nf : (diff == 0.0 ? 0.0 : INFINITY);
      if (L.perr) eps = NAN;   // the two-wave sweep lost its count: stop and report eps = NaN
      L.stop = (eps <= tol || L.perr) ? 1 : 0;
      L.red[0] = bpart * (1.0 + 1e-12);
    }
    __syncthreads();
    const double Bb = L.red[0];
    // ---- verify the skipped contacts
    for (int c = tid; c < nc; c += PGS_NT) {
      if (L.inS[c]) continue;
      const double g = gnSet[c], rb = swn[c] * Bb;
      if (!(g - rb > 1e-13 * (fabs(g) + rb))) L.ulist[atomicAdd(&L.nu, 1)] = (unsigned short)c;
    }
    __syncthreads();
    const int nu = L.nu;
    for (int u = wv; u < nu; u += PGS_NW) {
      const int c = L.ulist[u];
      double pt[3];
      pca_turn_proximity(c, nS, m, WH, Pset, h2, L, ln, pt);
      if (ln == 0) {
        const double ps[3] = {pstart[3 * c], pstart[3 * c + 1], pstart[3 * c + 2]};
        double F[3][3], delta[3];
        contact_frame(obs, t0, t1, pt, ps, F, delta);
        if (delta[0] < 0.0) {
          L.inS[c] = 1;
          L.flag = 1;
        }
      }
    }
    __syncthreads();
    if (L.flag && !L.perr) {
      // a skipped contact was not a no-op: restart the sweep with a larger S
      for (int r = tid; r < 3 * nS; r += PGS_NT) f[3L * L.Sidx[r / 3] + r % 3] = L.f0[r];
      need_build = true;
      __threadfence_block();
      __syncthreads();
      continue;
    }
    ++sweep;
    if (L.stop) break;
  }
  // ---- results: S from its records; the others separate, with the frame at
  // their proximity at their turn in the last sweep
  for (int r = tid; r < 3 * nS; r += PGS_NT) {
    const long e = 3L * L.Sidx[r / 3] + r % 3;
    const double *rc = L.rec + PCA_RW * (r / 3);
    f[e] = rc[22 + r % 3];
    lam[e] = rc[10 + r % 3];
  }
  for (int i = tid; i < nS; i += PGS_NT) {
    const double *rc = L.rec + PCA_RW * i;
    for (int q = 0; q < 9; ++q) C[9L * L.Sidx[i] + q] = rc[13 + q];
    status[L.Sidx[i]] = (int8_t)L.stS[i];
  }
  for (int c = wv; c < nc; c += PGS_NW) {
    if (L.inS[c]) continue;
    double pt[3];
    pca_turn_proximity(c, nS, m, WH, Pset, h2, L, ln, pt);
    if (ln == 0) {
      const double ps[3] = {pstart[3 * c], pstart[3 * c + 1], pstart[3 * c + 2]};
      double F[3][3], delta[3];
      contact_frame(obs, t0, t1, pt, ps, F, delta);
      for (int r = 0; r < 3; ++r) {
        for (int q = 0; q < 3; ++q) C[9L * c + 3 * r + q] = F[r][q];
        lam[3 * c + r] = 0.0;
      }
      status[c] = (int8_t)ICR_SEPARATE;
    }
  }
  if (tid == 0) {
    *sweeps_out = sweep;
    *eps_out = eps;
  }
}

// ---- large active sets: block Gauss-Seidel over the whole GPU --------------
//
// When the active set outgrows the register chains (k_pgs_active hands over
// with ctl[0] = 1 and the sweep to resume in ctl[1]), the remaining sweeps
// run here, with the iterates of the sequential sweep: the contacts are
// taken in blocks of 128 in index order, and every block's force changes
// reach the gaps of all contacts, g += W~[:, block] dlambda (rows of the
// exactly symmetric W stand for its columns), before those contacts' turn.
// One cooperative launch with no grid barrier inside the sweeps:
//  - workgroup 0 (the lead) runs the chain of a block in waves 0 and 1 (the
//    chains of the active-set kernel, 64 contacts each; contacts that stay
//    separated are passed over); meanwhile waves 2-7 stage the next block's
//    records and forces in the other half of the LDS arrays and add the
//    block's force changes to the gaps of the NEXT block as the chain
//    publishes them.  So the next chain starts without waiting for the rest
//    of the GPU.
//  - the other workgroups push each published block's changes into all other
//    gap rows (64-row chunks, each chunk always owned by the same workgroup),
//    one block behind the lead, and report the last block they finished.
// The lead reads the next block's gaps only after every pushing workgroup
// finished the block before the current one, and reuses a block's change
// list (double-buffered) only after all of them read it.  Launched only when
// the stream is not being captured (else k_pgs_single continues).
constexpr int COOP_B = kPgsCoopB;   // contacts per block
constexpr int COOP_NT = PGS_NT;     // threads per workgroup
constexpr int COOP_MAXG = 128;      // workgroups of the launch at most
static_assert(3 * COOP_B == 6 * 64, "a block's gap rows are six 64-row chunks");
static_assert(COOP_NT == 512, "lead workgroup: two chain waves, six follower waves");
// sync words: [0] last published block, [1] stop, [2..3] changed contacts per
// list buffer, [4] a wait gave up, [8 + w] last block pushed by workgroup w
constexpr int COOP_SYNC_PUB = 0, COOP_SYNC_STOP = 1, COOP_SYNC_CNT = 2, COOP_SYNC_ERR = 4, COOP_SYNC_PROG = 8;
// Every wait is bounded (polls of device memory / of LDS, seconds in all,
// far beyond any legitimate wait): a wait that gives up sets the error word,
// every workgroup stops, and the call reports eps = NaN (not converged).
constexpr int COOP_SPIN_DEV = 1 << 22, COOP_SPIN_LDS = 1 << 24;
static_assert(COOP_SYNC_PROG + COOP_MAXG <= kPgsCoopSync, "sync words");
struct CoopArgs {
  int nc;
  const void *W;
  const double *d, *mu;
  double h2;
  double *lam;
  int8_t *status;
  int max_sweeps;
  double tol;
  int j_inner;
  int *sweeps_out;
  double *eps_out;
  const int *ctl;    // [0] handover, [1] first sweep
  double *g;         // [3 nc] gaps with the own term
  double *recAll;    // [PGS_RW][nc] records, then the entries w00 w01 w02 w11 w12 w22 of the blocks
  double *Wblk;      // [nblocks * COOP_B * COOP_B * PGS_BLK] blocked diagonal couplings
  double *dl;        // [2][3 COOP_B] force changes of the last two blocks
  int *chg;          // [2][COOP_B] their changed contacts (block-local)
  int *sync;         // [kPgsCoopSync] sync words
};

// Loads of data another workgroup of the launch wrote go to the
// device-coherent level, past this compute unit's own cache.
__device__ inline double ld_dev(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int ld_dev(const int *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void st_dev(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline int ld_wg(const int *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
__device__ inline void st_wg(int *p, int v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// y[r] = base[r] + h2 sum_k sum_a M[(3 c_k + a) m + r] v[3 k + a] for the rows
// of the 64-row chunks first, first + stride, ... outside [skip_lo, skip_hi):
// wave v takes list entries v, v + 8, ... (four at a time, twelve loads in
// flight); the eight partial sums are added in wave order.  W streams
// through with non-temporal loads, so that it does not evict the blocked
// couplings the chain reads.
template <class TW>
__device__ void coop_rows(int m, const TW *__restrict__ M, const unsigned short *list, int nlist, const double *vals,
                          int cbase, const double *base, double h2, double *y, double *part, int first, int stride,
                          int skip_lo, int skip_hi) {
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  constexpr int NW = COOP_NT / 64;
  const int nchunk = (m + 63) / 64;
  for (int ch = first; ch < nchunk; ch += stride) {
    if (ch >= skip_lo && ch < skip_hi) continue;
    const int r = 64 * ch + ln;
    double a = 0.0;
    if (r < m) {
      for (int k = wv; k < nlist; k += 4 * NW) {
        double x[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int kk = k + NW * q;
          const long c3 = 3L * (cbase + list[kk < nlist ? kk : k]);
#pragma unroll
          for (int t = 0; t < 3; ++t) x[q][t] = kk < nlist ? (double)__builtin_nontemporal_load(M + (c3 + t) * m + r) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int kk = k + NW * q;
          if (kk < nlist) {
            const double *vk = vals + 3 * kk;
            a = fma(x[q][0], vk[0], a);
            a = fma(x[q][1], vk[1], a);
            a = fma(x[q][2], vk[2], a);
          }
        }
      }
    }
    part[wv * 64 + ln] = a;
    __syncthreads();
    if (wv == 0 && r < m) {
      double t = 0.0;
      for (int w = 0; w < NW; ++w) t += part[w * 64 + ln];
      y[r] = ld_dev(base + r) + h2 * t;
    }
    __syncthreads();
  }
}

// Own-term-free gap of row e of the block staged at contact o of the LDS
// arrays: g - w lambda, w the contact's 3x3 block (the record's last six rows,
// w00 w01 w02 w11 w12 w22), lambda its current force.
__device__ inline double coop_own_free(const PgsLds &L, int o, int e, double g) {
  const int c = o + e / 3, r = e % 3;
  const double *w = L.rec + PGS_RC * PGS_SMAX + c;
  const double w0 = w[(r == 0 ? 0 : r == 1 ? 1 : 2) * PGS_SMAX];
  const double w1 = w[(r == 0 ? 1 : r == 1 ? 3 : 4) * PGS_SMAX];
  const double w2 = w[(r == 0 ? 2 : r == 1 ? 4 : 5) * PGS_SMAX];
  return g - (w0 * L.lamS[3 * c] + w1 * L.lamS[3 * c + 1] + w2 * L.lamS[3 * c + 2]);
}

// Lead workgroup (see above).
template <class TW>
__device__ void coop_lead(const CoopArgs &a, PgsLds &L, int sweep0) {
  const TW *__restrict__ W = static_cast<const TW *>(a.W);
  const int nc = a.nc, m = 3 * nc, nb = (nc + COOP_B - 1) / COOP_B;
  const double h2 = a.h2;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const long blk_elems = (long)COOP_B * COOP_B * PGS_BLK;
  const int G = gridDim.x;
  const int total = (a.max_sweeps - sweep0) * nb;   // blocks to sweep
  int sweep = sweep0;
  double eps = 0.0;
  if (total > 0) {
    // block 0 staged at contact 0 of the LDS arrays
    {
      const int nB = min(COOP_B, nc);
      for (int e = tid; e < nB * PGS_RW; e += COOP_NT)
        L.rec[PGS_SMAX * (e / nB) + e % nB] = a.recAll[(long)nc * (e / nB) + e % nB];
      for (int e = tid; e < 3 * nB; e += COOP_NT) L.lamS[e] = L.lamS0[e] = a.lam[e];
      __syncthreads();
      for (int e = tid; e < 3 * nB; e += COOP_NT) L.gS[e] = coop_own_free(L, 0, e, ld_dev(a.g + e));
      if (tid == 0) {
        L.cprog = 0;
        L.cflag = 0;
        L.stop = 0;
        L.perr = 0;
      }
      __syncthreads();
    }
    const int wu = __builtin_amdgcn_readfirstlane(wv);
    double dsum = 0.0, nl2 = 0.0;   // wave 0: sums of the sweep
    for (int s = 0; s < total; ++s) {
      const int b = s % nb, bn = (b + 1) % nb, p = s & 1;
      const int o = p ? COOP_B : 0, o1 = COOP_B - o;
      const int c0 = COOP_B * b, nB = min(COOP_B, nc - c0), nsp = pgs_wave_pad(nB);
      const int cn0 = COOP_B * bn, nBn = min(COOP_B, nc - cn0);
      // waves 0-1: the chain of this block, each over its 64 contacts
      if (64 * wu < min(nB, 128)) {
        const BlkBuf buf(a.Wblk + (long)b * blk_elems, 8u * PGS_BLK * (unsigned)nsp * (unsigned)nB);
        const int me = o + 64 * wu + ln;
        const bool on = 64 * wu + ln < nB;
        ChainLane c;
        c.rc = pgs_rec_load(L, on ? me : o);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          c.e[q] = on ? L.gS[3 * me + q] : 0.0;
          c.l[q] = on ? L.lamS[3 * me + q] : 0.0;
        }
        if (a.j_inner == 8)
          chain_sweep<8, true>(c, nB, nsp, buf, o, 0, L, a.j_inner, wu, ln);
        else
          chain_sweep<0, true>(c, nB, nsp, buf, o, 0, L, a.j_inner, wu, ln);
        if (on) L.stS[me] = (unsigned char)c.st;
      }
      // waves 2-7: row f of the next block, f < 3 nBn
      const bool follower = wv >= 2;
      const int f = 64 * (wv - 2) + ln;
      double acc = 0.0, gold = 0.0;
      bool have_g = false;
      if (follower) {
        const bool act = f < 3 * nBn;
        const long row = 3L * cn0 + (act ? f : 0);
        // W~ rows of four contacts at a time, the next four in flight
        auto load = [&](double (&x)[4][3], int i) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const long c3 = 3L * (c0 + min(i + q, nB - 1));
#pragma unroll
            for (int t = 0; t < 3; ++t) x[q][t] = (double)__builtin_nontemporal_load(W + (c3 + t) * m + row);
          }
        };
        double x[2][4][3];
        load(x[0], 0);
        load(x[1], 4);
        // stage the next block's records and forces (unchanged by this chain)
        for (int e = f; e < nBn * PGS_RW; e += COOP_NT - 128)
          L.rec[PGS_SMAX * (e / nBn) + o1 + e % nBn] = a.recAll[(long)nc * (e / nBn) + cn0 + e % nBn];
        if (act) L.lamS[3 * o1 + f] = L.lamS0[3 * o1 + f] = a.lam[3 * cn0 + f];
        if (wv == 7) {
          // every pushing workgroup finished block s - 1: the next block's gap
          // rows hold all earlier changes, and list buffer p ^ 1 is free
          for (int spin = 0;; ++spin) {
            bool ok = true;
            for (int w = 1 + ln; w < G; w += 64) ok &= ld_dev(a.sync + COOP_SYNC_PROG + w) >= s - 1;
            if (__ballot(!ok) == 0ull) break;
            if (spin == COOP_SPIN_DEV) {
              if (ln == 0) st_dev(a.sync + COOP_SYNC_ERR, 1);
              break;
            }
            __builtin_amdgcn_s_sleep(2);
          }
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          if (ln == 0) st_wg(&L.cflag, 1);
        }
        for (int i = 0; i < nB; i += 8) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int ih = i + 4 * h;
            if (ih < nB) {
              const int need = min(ih + 4, nB);
              for (int spin = 0; ld_wg(&L.cprog) < need; ++spin) {
                if (spin == COOP_SPIN_LDS) {
                  st_dev(a.sync + COOP_SYNC_ERR, 1);
                  break;
                }
                __builtin_amdgcn_s_sleep(1);
              }
              __atomic_signal_fence(__ATOMIC_SEQ_CST);
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                if (ih + q < nB) {
                  const double *l = L.lamS + 3 * (o + ih + q), *l0 = L.lamS0 + 3 * (o + ih + q);
                  acc = fma(x[h][q][0], l[0] - l0[0], acc);
                  acc = fma(x[h][q][1], l[1] - l0[1], acc);
                  acc = fma(x[h][q][2], l[2] - l0[2], acc);
                }
              }
              load(x[h], ih + 8);
            }
          }
          if (!have_g && ld_wg(&L.cflag) != 0) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            gold = act ? ld_dev(a.g + row) : 0.0;
            have_g = true;
          }
        }
        if (!have_g) {
          for (int spin = 0; ld_wg(&L.cflag) == 0; ++spin) {
            if (spin == COOP_SPIN_LDS) {
              st_dev(a.sync + COOP_SYNC_ERR, 1);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          gold = act ? ld_dev(a.g + row) : 0.0;
        }
      }
      __syncthreads();
      if (wv == 0) {
        // new forces and statuses out, the changed contacts listed
        int cnt = 0;
        for (int i0 = 0; i0 < nB; i0 += 64) {
          const int i = i0 + ln;
          double d0 = 0.0, d1 = 0.0, d2 = 0.0, q2 = 0.0;
          if (i < nB) {
            const double *l = L.lamS + 3 * (o + i), *l0 = L.lamS0 + 3 * (o + i);
            d0 = l[0] - l0[0];
            d1 = l[1] - l0[1];
            d2 = l[2] - l0[2];
            q2 = l[0] * l[0] + l[1] * l[1] + l[2] * l[2];
            a.lam[3 * (c0 + i)] = l[0];
            a.lam[3 * (c0 + i) + 1] = l[1];
            a.lam[3 * (c0 + i) + 2] = l[2];
            a.status[c0 + i] = (int8_t)L.stS[o + i];
          }
          const bool ch = (d0 != 0.0) | (d1 != 0.0) | (d2 != 0.0);
          const unsigned long long bal = __ballot(ch);
          if (ch) {
            const int k = cnt + __popcll(bal & ((1ull << ln) - 1ull));
            a.chg[COOP_B * p + k] = i;
            a.dl[3 * COOP_B * p + 3 * k] = d0;
            a.dl[3 * COOP_B * p + 3 * k + 1] = d1;
            a.dl[3 * COOP_B * p + 3 * k + 2] = d2;
          }
          cnt += __popcll(bal);
          double sq = d0 * d0 + d1 * d1 + d2 * d2;
          for (int w = 32; w > 0; w >>= 1) {
            sq += __shfl_xor(sq, w, 64);
            q2 += __shfl_xor(q2, w, 64);
          }
          dsum += sq;   // same order every time
          nl2 += q2;
        }
        if (ln == 0) a.sync[COOP_SYNC_CNT + p] = cnt;
        int stop = 0;
        if (b == nb - 1) {
          // end of the sweep: eps = |lambda_i - lambda_{i-1}| / |lambda_i|
          const double diff = sqrt(dsum), nl = sqrt(nl2);
          eps = nl > 0.0 ? diff / nl : (diff == 0.0 ? 0.0 : INFINITY);
          ++sweep;
          stop = (eps <= a.tol || sweep >= a.max_sweeps) ? 1 : 0;
          dsum = nl2 = 0.0;
        }
        if (L.perr && ln == 0) st_dev(a.sync + COOP_SYNC_ERR, 1);   // the chain's waves lost their count
        if (L.perr || ld_dev(a.sync + COOP_SYNC_ERR) != 0) stop = 1;
        if (ln == 0) {
          L.stop = stop;
          if (stop) a.sync[COOP_SYNC_STOP] = 1;
        }
      } else if (follower && f < 3 * nBn) {
        const double gn = gold + h2 * acc;
        a.g[3L * cn0 + f] = gn;
        L.gS[3 * o1 + f] = coop_own_free(L, o1, f, gn);
      }
      __threadfence();
      if (tid == 0) {
        L.cprog = 0;
        L.cflag = 0;
      }
      __syncthreads();
      if (tid == 0) st_dev(a.sync + COOP_SYNC_PUB, s);
      if (L.stop) break;
    }
  } else if (tid == 0) {
    a.sync[COOP_SYNC_STOP] = 1;
    __threadfence();
    st_dev(a.sync + COOP_SYNC_PUB, 0);
  }
  if (tid == 0) {
    *a.sweeps_out = sweep;
    if (ld_dev(a.sync + COOP_SYNC_ERR) != 0)
      *a.eps_out = NAN;
    else if (total > 0)
      *a.eps_out = eps;
  }
}

// Pushing workgroups: block s's changes into every owned chunk of gap rows
// outside the next block, in block order, until the lead stops.
template <class TW>
__device__ void coop_push(const CoopArgs &a, PgsLds &L) {
  const TW *__restrict__ W = static_cast<const TW *>(a.W);
  const int nc = a.nc, m = 3 * nc, nb = (nc + COOP_B - 1) / COOP_B;
  const int tid = threadIdx.x;
  const int G = gridDim.x;
  for (int s = 0;; ++s) {
    if (tid == 0) {
      int stop = 0;
      for (int spin = 0; ld_dev(a.sync + COOP_SYNC_PUB) < s && (stop = ld_dev(a.sync + COOP_SYNC_STOP)) == 0; ++spin) {
        if (spin == COOP_SPIN_DEV) {
          st_dev(a.sync + COOP_SYNC_ERR, 1);
          stop = 1;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      if (!stop) stop = ld_dev(a.sync + COOP_SYNC_STOP);
      L.stop = stop;
    }
    __syncthreads();
    if (L.stop) break;
    const int b = s % nb, bn = (b + 1) % nb, p = s & 1;
    const int nchg = ld_dev(a.sync + COOP_SYNC_CNT + p);
    for (int e = tid; e < nchg; e += COOP_NT) L.ulist[e] = (unsigned short)ld_dev(a.chg + COOP_B * p + e);
    for (int e = tid; e < 3 * nchg; e += COOP_NT) L.lamSet[e] = ld_dev(a.dl + 3 * COOP_B * p + e);
    __syncthreads();
    if (nchg > 0)
      coop_rows<TW>(m, W, L.ulist, nchg, L.lamSet, COOP_B * b, a.g, a.h2, a.g, L.lamS, blockIdx.x - 1, G - 1, 6 * bn,
                    6 * bn + 6);
    __threadfence();
    __syncthreads();
    if (tid == 0) st_dev(a.sync + COOP_SYNC_PROG + blockIdx.x, s);
  }
}

template <class TW>
__global__ __launch_bounds__(COOP_NT) void k_pgs_coop(CoopArgs a) {
  extern __shared__ double lds_raw[];
  PgsLds &L = *reinterpret_cast<PgsLds *>(lds_raw);
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  // control words written by the active-set kernel (an earlier launch)
  if (a.ctl[0] == 0) return;   // uniform: the active-set kernel finished the call
  const int sweep0 = a.ctl[1];
  const TW *__restrict__ W = static_cast<const TW *>(a.W);
  const int nc = a.nc, m = 3 * nc;
  const double h2 = a.h2;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const int nb = (nc + COOP_B - 1) / COOP_B;
  const long blk_elems = (long)COOP_B * COOP_B * PGS_BLK;
  const long gthreads = (long)gridDim.x * COOP_NT, gt = (long)blockIdx.x * COOP_NT + tid;
  // ---- set-up, all workgroups: sync words, records, blocked couplings, gaps
  // at the resume state
  if (gt < kPgsCoopSync)
    a.sync[gt] = (gt == COOP_SYNC_STOP || gt == COOP_SYNC_CNT || gt == COOP_SYNC_CNT + 1 || gt == COOP_SYNC_ERR) ? 0 : -1;
  for (long c = gt; c < nc; c += gthreads) {
    double wb[3][3];
    for (int p = 0; p < 3; ++p)
      for (int q = 0; q < 3; ++q) wb[p][q] = h2 * (double)W[(3 * c + p) * m + 3 * c + q];
    const PgsRec tmp = make_record(wb, a.mu[c]);
    const double *x = reinterpret_cast<const double *>(&tmp);
    for (int q = 0; q < PGS_RC; ++q) a.recAll[(long)q * nc + c] = x[q];
    const double bw[6] = {wb[0][0], wb[0][1], wb[0][2], wb[1][1], wb[1][2], wb[2][2]};
    for (int q = 0; q < 6; ++q) a.recAll[(long)(PGS_RC + q) * nc + c] = bw[q];
  }
  for (long e = gt; e < (long)nb * blk_elems; e += gthreads) {
    const int b = (int)(e / blk_elems);
    const long r = e % blk_elems;
    const int c0 = COOP_B * b, nB = min(COOP_B, nc - c0), nsp = pgs_wave_pad(nB);
    const int per = nsp * PGS_BLK, i = (int)(r / per), rr = (int)(r % per);
    int l, j;
    blk_index(rr % BLK_GROUP, l, j);
    const int c = 64 * (rr / BLK_GROUP) + l;
    if (i >= nB) continue;
    double v = 0.0;
    if (c < nB && c != i) v = h2 * (double)W[(3L * (c0 + i) + j % 3) * m + 3L * (c0 + c) + j / 3];
    a.Wblk[e] = v;
  }
  {
    // contacts with a force, in every workgroup's LDS (order is fixed); the
    // running count is a wave-uniform register (the ballot is uniform)
    if (wv == 0) {
      int cnt = 0;
      for (int c0 = 0; c0 < nc; c0 += 64) {
        const int c = c0 + ln;
        const bool nz = c < nc && (a.lam[3 * c] != 0.0 || a.lam[3 * c + 1] != 0.0 || a.lam[3 * c + 2] != 0.0);
        const unsigned long long bal = __ballot(nz);
        if (nz) L.ulist[cnt + __popcll(bal & ((1ull << ln) - 1ull))] = (unsigned short)c;
        cnt += __popcll(bal);
      }
      if (ln == 0) L.nu = cnt;
    }
    __syncthreads();
    const int nl = L.nu;
    // the force values in the order of the list, in LDS (reuses the set's gap area)
    double *vals = L.lamSet;
    double *part = L.lamS;
    for (int q0 = 0; q0 < nl; q0 += PGS_S3 / 3) {
      const int nq = min(PGS_S3 / 3, nl - q0);
      for (int e = tid; e < 3 * nq; e += COOP_NT) vals[e] = a.lam[3 * L.ulist[q0 + e / 3] + e % 3];
      __syncthreads();
      coop_rows<TW>(m, W, L.ulist + q0, nq, vals, 0, q0 == 0 ? a.d : a.g, h2, a.g, part, blockIdx.x, gridDim.x, 0, 0);
    }
    if (nl == 0)
      for (long r = gt; r < m; r += gthreads) a.g[r] = a.d[r];
  }
  __threadfence();
  grid.sync();
  if (blockIdx.x == 0)
    coop_lead<TW>(a, L, sweep0);
  else
    coop_push<TW>(a, L);
}

__global__ void k_world_force(int nc, const double *__restrict__ C, const double *__restrict__ lam,
                              double *__restrict__ f) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 3 * nc) return;
  f[e] = world_force(C, lam, e / 3, e % 3);
}

__global__ void k_zero(long n, double *__restrict__ x) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) x[i] = 0.0;
}

// Warm start of the next step (one workgroup): clear the forces of the
// previous step's contact nodes (count and ids on the device), store this
// step's world-frame forces on their nodes, keep their ids, advance the time.
// Pair contacts (the first npair contacts) keep their own forces.
__global__ __launch_bounds__(1024) void k_store_forces(int nc, const int *__restrict__ nodes,
                                                       const double *__restrict__ f, double *__restrict__ node_force,
                                                       int *__restrict__ prev_nodes, int *__restrict__ prev_nc,
                                                       StepCtx *__restrict__ ctx, int npair,
                                                       const double *__restrict__ fpair_new,
                                                       double *__restrict__ fpair) {
  for (int e = threadIdx.x; e < 3 * npair; e += blockDim.x) fpair[e] = fpair_new[e];
  const int pn = *prev_nc;
  for (int c = threadIdx.x; c < pn; c += blockDim.x) {
    const int v = prev_nodes[c];
    for (int a = 0; a < 3; ++a) node_force[3 * v + a] = 0.0;
  }
  __syncthreads();
  for (int c = threadIdx.x; c < nc; c += blockDim.x) {
    const int v = nodes[c];
    for (int a = 0; a < 3; ++a) node_force[3 * v + a] = f[3 * c + a];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < nc; c += blockDim.x) prev_nodes[c] = nodes[c];
  if (threadIdx.x == 0) {
    *prev_nc = nc;
    ctx->t0 = ctx->t0 + ctx->h;
  }
}

// p = H q_k with q_k = q_free + h^2 A^-1 J^T lambda (Algorithm 2, steps 4-6).
__global__ void k_std_proximity(int nc, const int *__restrict__ nodes, const double *__restrict__ qf,
                                const double *__restrict__ sol, double h2, double *__restrict__ p) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nc) return;
  int v = nodes[c];
  for (int a = 0; a < 3; ++a) p[3 * c + a] = qf[3 * v + a] + h2 * sol[3 * v + a];
}

__global__ void k_set_ctx(StepCtx *ctx, icr_obstacle obs, int set_obs, double t0, int set_t, double h) {
  if (set_obs) ctx->obs = obs;
  if (set_t) ctx->t0 = t0;
  ctx->h = h;
}

__global__ void k_stamp(unsigned long long *ts, int slot) { ts[slot] = wall_clock64(); }


}  // namespace

void launch_select_contacts(icr_scene *s, int nc) {
  auto &C = s->con;
  const int P = s->pairs.count;   // pair contacts come first; the obstacle contacts follow them
  k_select<<<1, 1024, 0, s->stream>>>(C.count, C.d_cand, s->st.d_qfree, s->st.d_q, s->st.d_ctx, nc - P,
                                      C.d_mu_node, s->st.d_node_force, C.d_nodes_c + P, C.d_mu + P,
                                      C.d_pfree + 3L * P, C.d_pstart + 3L * P, C.d_f + 3L * P);
  ICR_LAUNCH_CHECK();
}

void launch_directions(icr_scene *s, int nc, bool first) {
  auto &C = s->con;
  const double *p = first ? C.d_pfree : C.d_p;
  k_directions<<<cdiv(nc, 128), 128, 0, s->stream>>>(nc, s->st.d_ctx, p, C.d_pfree, C.d_pstart, C.d_f, C.d_C,
                                                     C.d_dk, C.d_lam, s->pairs.count, s->pairs.d_normal);
  ICR_LAUNCH_CHECK();
}

// Pair contacts 0..P-1 of a step: p_free = H q_free, p_start = H q over their
// slots, friction, warm start from the pair's previous force, node id -1;
// and the node list of the W_H build: the pairs' distinct nodes, then the
// step's obstacle contact nodes (contacts P..nc-1).
__global__ void k_pair_points(int P, int nc, int nup, const int *__restrict__ slot_node,
                              const double *__restrict__ w, const double *__restrict__ qf,
                              const double *__restrict__ q, const double *__restrict__ mu_pair,
                              const double *__restrict__ fpair, const int *__restrict__ pair_nodes,
                              int *__restrict__ nodes_c, double *__restrict__ mu_c, double *__restrict__ pfree,
                              double *__restrict__ pstart, double *__restrict__ finit, int *__restrict__ unodes) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < P) {
    double a[3] = {0, 0, 0}, b[3] = {0, 0, 0};
    for (int k = 0; k < 4; ++k) {
      const int v = slot_node[4 * t + k];
      if (v < 0) continue;
      const double wk = w[4 * t + k];
      for (int x = 0; x < 3; ++x) {
        a[x] = fma(wk, qf[3 * v + x], a[x]);
        b[x] = fma(wk, q[3 * v + x], b[x]);
      }
    }
    for (int x = 0; x < 3; ++x) {
      pfree[3 * t + x] = a[x];
      pstart[3 * t + x] = b[x];
      finit[3 * t + x] = fpair[3 * t + x];
    }
    mu_c[t] = mu_pair[t];
    nodes_c[t] = -1;
  }
  if (t < nup) unodes[t] = pair_nodes[t];
  if (t >= nup && t < nup + nc - P) unodes[t] = nodes_c[P + t - nup];
}

// Force on every node of the W_H build (H_w^T f): a pair node sums weight x
// force over the pair slots that name it (CSR in slot order), an obstacle
// contact's node takes that contact's force.
__global__ void k_node_forces(int nup, int nu, int P, const int *__restrict__ csr_ptr,
                              const int *__restrict__ csr_slot, const double *__restrict__ w,
                              const double *__restrict__ f, double *__restrict__ fu) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nu) return;
  double a[3] = {0, 0, 0};
  if (u < nup) {
    for (int e = csr_ptr[u]; e < csr_ptr[u + 1]; ++e) {
      const int sl = csr_slot[e], c = sl / 4;
      for (int x = 0; x < 3; ++x) a[x] = fma(w[sl], f[3 * c + x], a[x]);
    }
  } else {
    const int c = P + u - nup;
    for (int x = 0; x < 3; ++x) a[x] = f[3 * c + x];
  }
  for (int x = 0; x < 3; ++x) fu[3 * u + x] = a[x];
}

void launch_pair_points(icr_scene *s, int nc) {
  auto &C = s->con;
  auto &Pr = s->pairs;
  const int n = std::max(Pr.count, Pr.nu + nc - Pr.count);
  k_pair_points<<<cdiv(n, 256), 256, 0, s->stream>>>(Pr.count, nc, Pr.nu, Pr.d_slot_node, Pr.d_w, s->st.d_qfree,
                                                     s->st.d_q, Pr.d_mu, Pr.d_force, Pr.d_nodes, C.d_nodes_c,
                                                     C.d_mu, C.d_pfree, C.d_pstart, C.d_f, Pr.d_unodes);
  ICR_LAUNCH_CHECK();
}

void launch_node_forces(icr_scene *s, int nc, const double *f, double *fu) {
  auto &Pr = s->pairs;
  const int nu = Pr.nu + nc - Pr.count;
  k_node_forces<<<cdiv(nu, 256), 256, 0, s->stream>>>(Pr.nu, nu, Pr.count, Pr.d_csr_ptr, Pr.d_csr_slot, Pr.d_w,
                                                      f, fu);
  ICR_LAUNCH_CHECK();
}

template <class TW>
void launch_update_W(hipStream_t st, int nc, const TW *WH, const double *Cm, TW *W) {
  long nb = (long)nc * nc;
  k_update_W<TW><<<(unsigned)((nb + 255) / 256), 256, 0, st>>>(nc, WH, Cm, W);
  ICR_LAUNCH_CHECK();
}
template void launch_update_W<double>(hipStream_t, int, const double *, const double *, double *);
template void launch_update_W<float>(hipStream_t, int, const float *, const double *, float *);

template <class TW>
void launch_pgs(hipStream_t st, int nc, const TW *W, const double *d, const double *mu, double h, double *lam,
                int8_t *status, int max_sweeps, double tol, int j_inner, int *sweeps_dev, double *eps_dev,
                const PgsWork &wk) {
  const int m = 3 * nc;
  // g0 = d + W~ lambda over the contacts with a warm-start force
  k_sym_gemv_sparse<TW><<<cdiv(m, 64), SG_NT, 0, st>>>(nc, W, d, lam, h * h, wk.g, nullptr, nullptr, nullptr);
  ICR_LAUNCH_CHECK();
  k_pgs_gather<TW><<<512, 256, 0, st>>>(nc, W, wk.g, lam, mu, h * h, wk.Sidx, wk.nS, wk.gnSet, wk.swn, wk.Wss, wk.rec,
                                    wk.gS);
  ICR_LAUNCH_CHECK();
  k_pgs_active<TW><<<1, PGS_NT, sizeof(PgsLds), st>>>(nc, W, d, wk.g, mu, h * h, lam, status, max_sweeps, tol, j_inner,
                                                sweeps_dev, eps_dev, wk.Wss, wk.gnSet, wk.swn, wk.ctl, wk.Sidx,
                                                wk.nS, wk.rec, wk.gS);
  ICR_LAUNCH_CHECK();
  // continues only if the active set outgrew the compact path: block
  // Gauss-Seidel over the whole GPU, or (under stream capture, or without
  // its buffers) the single-workgroup sweep
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  ICR_HIP(hipStreamIsCapturing(st, &cap));
  // One pushing workgroup to two chunks of gap rows at most: they poll and are
  // polled at device level, and more of them slow the lead's chain, while fewer
  // fall behind it.  Ten sweeps with every contact pressed and one, two, four
  // and eight chunks to a workgroup: 600 contacts 2.77, 2.79, 3.18, 3.88 ms;
  // 1000 4.75, 4.79, 5.39, 6.60; 1500 7.6, 7.5, 8.2, 10.5; 2200 12.1, 11.5,
  // 12.4, 15.7; 3000 19.5, 16.5, 17.4, 21.6.
  const int G = std::min(coop_grid(), 1 + cdiv(3L * nc, 128));
  if (nc > PGS_WAVE_MAX && wk.Wblk != nullptr && G > 1 && cap == hipStreamCaptureStatusNone) {
    CoopArgs a{nc, W, d, mu, h * h, lam, status, max_sweeps, tol, j_inner, sweeps_dev, eps_dev, wk.ctl, wk.g,
               wk.recAll, wk.Wblk, wk.dl, wk.chg, wk.csync};
    void *args[] = {&a};
    ICR_HIP(hipLaunchCooperativeKernel((const void *)k_pgs_coop<TW>, dim3(G), dim3(COOP_NT), args, sizeof(PgsLds), st));
  } else {
    k_pgs_single<TW><<<1, 1024, pgs_single_lds(nc), st>>>(nc, W, d, nullptr, mu, h * h, lam, status, max_sweeps, tol,
                                                          j_inner, sweeps_dev, eps_dev, wk.ctl);
    ICR_LAUNCH_CHECK();
  }
}
template void launch_pgs<double>(hipStream_t, int, const double *, const double *, const double *, double, double *,
                                 int8_t *, int, double, int, int *, double *, const PgsWork &);
template void launch_pgs<float>(hipStream_t, int, const float *, const double *, const double *, double, double *,
                                int8_t *, int, double, int, int *, double *, const PgsWork &);

void launch_pgs_per_constraint(hipStream_t st, int nc, const StepCtx *ctx, const double *WH, const double *pfree,
                               const double *p, const double *pstart, const double *mu, double h, double *f,
                               double *Cm, double *lam, int8_t *status, int max_sweeps, double tol, int j_inner,
                               int *sweeps_dev, double *eps_dev, const PgsWork &wk) {
  // the register chain over the contacts that can change, then (only if
  // their set outgrew the chain) the one-workgroup sweep from that state
  k_pgs_pca<<<1, PGS_NT, sizeof(PcaLds), st>>>(nc, ctx, WH, pfree, p, pstart, mu, h * h, f, Cm, lam, status,
                                               max_sweeps, tol, j_inner, sweeps_dev, eps_dev, wk.Wss, wk.g, wk.gnSet,
                                               wk.swn, wk.ctl);
  ICR_LAUNCH_CHECK();
  k_pgs_pc<<<1, 1024, pgs_pc_lds(nc), st>>>(nc, ctx, WH, wk.g, pstart, mu, h * h, f, Cm, lam, status, max_sweeps, tol,
                                           j_inner, sweeps_dev, eps_dev, wk.ctl);
  ICR_LAUNCH_CHECK();
}

namespace {
int g_coop_grid[64];   // per device: workgroups of the cooperative PGS launch (0 = not available)
}

int coop_grid() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  return g_coop_grid[dev];
}

void pgs_prepare() {
  // kernel attributes are set once per device
  static std::mutex mtx;
  static unsigned long long done = 0;
  int dev = 0;
  ICR_HIP(hipGetDevice(&dev));
  const unsigned long long bit = 1ull << (dev & 63);
  std::lock_guard<std::mutex> lock(mtx);
  if (done & bit) return;
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_active<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(PgsLds)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_active<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(PgsLds)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_single<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pgs_single_lds(PGS_MAX_NC)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_single<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pgs_single_lds(PGS_MAX_NC)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_pc, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)pgs_pc_lds(PGS_MAX_NC)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_coop<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(PgsLds)));
  for (const void *f : {(const void *)k_batch_pgs, (const void *)k_batch_small})
    ICR_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(PgsLds)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_pca, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(PcaLds)));
  ICR_HIP(hipFuncSetAttribute((const void *)k_pgs_coop<float>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)sizeof(PgsLds)));
  // cooperative launch: at most one workgroup per compute unit (its LDS),
  // 128 workgroups at most (enough to stream the gap updates)
  int coop = 0, cus = 0, per_cu = 0;
  g_coop_grid[dev & 63] = 0;
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) == hipSuccess && coop &&
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)k_pgs_coop<double>, COOP_NT,
                                                   sizeof(PgsLds)) == hipSuccess &&
      per_cu > 0)
    g_coop_grid[dev & 63] = std::min(128, per_cu * cus);
  done |= bit;
}

void launch_newton_batch(hipStream_t st, const NewtonTask *tasks, const NewtonBatchIdx &ids, int max_nc, int wide,
                         int max_newton) {
  if (ids.n < 1 || ids.n > kNewtonBatchMax) throw std::runtime_error("batched Newton loop: 1..64 scenes");
  pgs_prepare();
  const int nc = max_nc;
  const dim3 one(1, ids.n), rows(cdiv(3L * nc, 64), ids.n);
  for (int k = 0; k < wide; ++k) {
    k_batch_directions<<<dim3(cdiv(nc, 128), ids.n), 128, 0, st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
    k_batch_update_W<<<dim3(cdiv((long)nc * nc, 256), ids.n), 256, 0, st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
    k_batch_gaps<<<rows, SG_NT, 0, st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
    k_batch_gather<<<dim3(std::max(32, 512 / ids.n), ids.n), 256, 0, st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
    k_batch_pgs<<<one, PGS_NT, sizeof(PgsLds), st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
    k_batch_proximity<<<rows, SG_NT, 0, st>>>(tasks, ids, k);
    ICR_LAUNCH_CHECK();
  }
  if (wide < max_newton) {
    k_batch_small<<<one, PGS_NT, sizeof(PgsLds), st>>>(tasks, ids, wide);
    ICR_LAUNCH_CHECK();
  }
}

void launch_world_force(hipStream_t st, int nc, const double *Cm, const double *lam, double *f) {
  k_world_force<<<cdiv(3 * nc, 256), 256, 0, st>>>(nc, Cm, lam, f);
  ICR_LAUNCH_CHECK();
}

template <class TW>
void launch_world_force_proximity(hipStream_t st, int nc, const double *Cm, const double *lam, double *f,
                                  const TW *WH, const double *p_free, double h, double *p) {
  const int m = 3 * nc;
  // f = C^T lambda and p = p_free + h^2 W_H f in one launch
  k_sym_gemv_sparse<TW><<<cdiv(m, 64), SG_NT, 0, st>>>(nc, WH, p_free, nullptr, h * h, p, Cm, lam, f);
  ICR_LAUNCH_CHECK();
}
template void launch_world_force_proximity<double>(hipStream_t, int, const double *, const double *, double *,
                                                   const double *, const double *, double, double *);
template void launch_world_force_proximity<float>(hipStream_t, int, const double *, const double *, double *,
                                                  const float *, const double *, double, double *);

template <class TW>
void launch_proximity(hipStream_t st, int nc, const TW *WH, const double *p_free, const double *f, double h,
                      double *p) {
  const int m = 3 * nc;
  // p = p_free + h^2 W_H f; f is zero at separated contacts
  k_sym_gemv_sparse<TW><<<cdiv(m, 64), SG_NT, 0, st>>>(nc, WH, p_free, f, h * h, p, nullptr, nullptr, nullptr);
  ICR_LAUNCH_CHECK();
}
template void launch_proximity<double>(hipStream_t, int, const double *, const double *, const double *, double,
                                       double *);
template void launch_proximity<float>(hipStream_t, int, const float *, const double *, const double *, double,
                                      double *);

void launch_set_ctx(icr_scene *s, const icr_obstacle *obs, const double *t0) {
  icr_obstacle o{};
  if (obs) o = *obs;
  k_set_ctx<<<1, 1, 0, s->stream>>>(s->st.d_ctx, o, obs ? 1 : 0, t0 ? *t0 : 0.0, t0 ? 1 : 0, s->mesh.h);
  ICR_LAUNCH_CHECK();
}

void launch_stamp(icr_scene *s, int slot) {
  k_stamp<<<1, 1, 0, s->stream>>>(s->st.d_stamps, slot);
  ICR_LAUNCH_CHECK();
}

void launch_standard_proximity(icr_scene *s, int nc) {
  const double h = s->mesh.h;
  k_std_proximity<<<cdiv(nc, 128), 128, 0, s->stream>>>(nc, s->con.d_nodes_c, s->st.d_qfree, s->st.d_sol, h * h,
                                                         s->con.d_p);
  ICR_LAUNCH_CHECK();
}

void launch_store_forces(icr_scene *s, int nc) {
  auto &S = s->st;
  const int P = s->pairs.count;
  k_store_forces<<<1, 1024, 0, s->stream>>>(nc - P, s->con.d_nodes_c + P, s->con.d_f + 3L * P, S.d_node_force,
                                            S.d_prev_nodes, S.d_prev_nc, S.d_ctx, P, s->con.d_f,
                                            s->pairs.d_force);
  ICR_LAUNCH_CHECK();
}

}  // namespace icr
