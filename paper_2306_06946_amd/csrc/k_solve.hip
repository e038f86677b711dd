// Solves against the supernodal factor P A P^T = L L^T.
//
// Multi-RHS (W_H = H A^-1 H^T, Eq. 28): with Z = L^{-1} P H^T,
// W_H = Z^T Z.  Contacts are sorted by the postorder index of the supernode
// holding their node, so the contacts below supernode s form one contiguous
// range [lo_s, hi_s) and its RHS front X_s has 3 (hi_s - lo_s) columns.  Per
// height level, bottom-up:
//   X_s  = unit columns of its own contacts, children's updates
//   Z_s  = L_ss^{-1} X_s[:n_s]                   (triangular dense product)
//   X_parent[rows below s] = X_s[n_s:] - L_21 Z_s
// then Wp = Z^T Z over the supernodes that two contacts share, and W_H is read
// out of it in contact order (exactly symmetric).
//
// Single RHS (free motion, corrective motion): the same forward sweep with one
// dense column, then the backward sweep top-down
//   x_s = L_ss^{-T} (y_s - L_21^T x[below rows of s]).
#include <algorithm>

#include "scene.hpp"

namespace icr {

namespace {

// ---- contact ordering -------------------------------------------------------

// Sort the contacts by (supernode, node, index): SORT_C contacts per
// workgroup, each one's place being the number of smaller packed 64-bit keys
// (they are distinct), counted by 16 waves over a sixteenth of the keys in LDS
// each.  (A bitonic network in one workgroup took 10, 19 and 61 us for 200,
// 1000 and 3000 contacts, this 5, 8 and 18.)  Invalid ids (out of range, clamped)
// get the key nsup, outside every supernode range, and duplicates are flagged;
// both make the call fail on the host.
constexpr int SORT_C = 64;
__global__ __launch_bounds__(1024) void k_sort_contacts(int nc, int N, int nsup, const int *__restrict__ node_ids,
                                                        const int *__restrict__ sup_of_node,
                                                        const uint8_t *__restrict__ fixed,
                                                        int *__restrict__ keys_sorted, int *__restrict__ order,
                                                        int *__restrict__ pos, int *__restrict__ cerr) {
  __shared__ unsigned long long kv[8192];
  __shared__ int part[16][SORT_C];
  const int tid = threadIdx.x, ln = tid & 63, wv = tid >> 6;
  for (int i = tid; i < nc; i += 1024) {
    const int node = node_ids[i];
    unsigned long long key = (unsigned long long)nsup, nd = 0;
    if (node < 0 || node >= N || fixed[node]) {
      atomicMax(cerr, 1);
    } else {
      key = (unsigned long long)sup_of_node[node];
      nd = (unsigned long long)node;
    }
    kv[i] = (key << 37) | (nd << 13) | (unsigned long long)i;
  }
  __syncthreads();
  const int i = SORT_C * blockIdx.x + ln;
  const unsigned long long mine = i < nc ? kv[i] : 0ull;
  const int per = (nc + 15) / 16, j1 = min(nc, (wv + 1) * per);
  int below = 0;
  bool twin = false;
#pragma unroll 4
  for (int j = wv * per; j < j1; ++j) {
    const unsigned long long v = kv[j];   // one key for the whole wave
    below += v < mine ? 1 : 0;
    twin |= (v >> 13) == (mine >> 13) && v != mine;
  }
  part[wv][ln] = below;
  if (twin && i < nc && (int)(mine >> 37) < nsup) atomicMax(cerr, 2);
  __syncthreads();
  if (wv == 0 && i < nc) {
    int p = 0;
    for (int w = 0; w < 16; ++w) p += part[w][ln];
    order[p] = i;
    keys_sorted[p] = (int)(mine >> 37);
    pos[i] = p;
  }
}

__device__ inline int lower_bound_i(const int *a, int n, int x) {
  int lo = 0, hi = n;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] < x)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

enum { RT_ASM = 0, RT_DIAG = 1, RT_OFF = 2, RHS_KINDS = 3 };

// Tile edges of the multi-RHS products.  A level's list of one kind is cut
// into 32 x 32 tiles if it has fewer than RHS_SMALL tiles of 64 x 64 and into
// 64 x 64 tiles otherwise; every entry is the same sum in the same order of k
// in both.  A short list leaves compute units idle while a workgroup spends
// 0.85 us of matrix time on 32 k of a 64 x 64 tile: the product of the root's
// 630 columns with 600 columns took 38 us in 100 tiles of 64 and takes 18 us in
// 380 of 32.  Lines at 256 and 1024 were 1 % slower at 1000 and 3000 contacts.
constexpr int RHS_T = 64, RHS_TS = 32;
constexpr int RHS_SMALL = 512;

// Tasks of one kind of one supernode with r RHS columns, n3 DOF columns and
// b3 below rows, for tiles of edge T: set X up (4 columns per task), L_ss^{-1}
// X (row tile x column tile), L_21 Z (below-row tile x column tile).  The host
// evaluates the same counts at r = rmax for the list capacities.
__host__ __device__ inline int rhs_task_count(int kind, int r, int n3, int b3, int T) {
  if (r <= 0) return 0;
  if (kind == RT_ASM) return (r + 3) / 4;
  return ((kind == RT_DIAG ? n3 : b3) + T - 1) / T * ((r + T - 1) / T);
}

// Order of tiles: bands of RHS_BAND columns (rows for Z^T Z) of tiles, across
// the band first, so that tiles that follow one another share panels of both
// operands.
constexpr int RHS_BAND = 8;
// u-th tile of a grid with nr rows and nc columns
__device__ inline void band_index(int u, int nr, int nc, int &i, int &j) {
  const int b = u / (RHS_BAND * nr), v = u - b * RHS_BAND * nr;
  const int w = min(RHS_BAND, nc - RHS_BAND * b);
  i = v / w;
  j = RHS_BAND * b + v % w;
}
// u-th tile of the lower triangle of an n x n grid
__device__ inline void band_tri_index(int u, int n, int &i, int &j) {
  int bi, bj;
  tri_index(u, bi, bj);
  const int b = bi / RHS_BAND, r0 = RHS_BAND * b;
  const int v = u - r0 * (r0 + 1) / 2, h = min(RHS_BAND, n - r0);
  if (v < h * r0) {
    i = r0 + v % h;
    j = v / h;
  } else {
    tri_index(v - h * r0, i, j);
    i += r0;
    j += r0;
  }
}

// k_rhs_plan (one workgroup per height level and kind): the contact range
// [lo, own, hi) of every supernode of the level (contacts are sorted by
// supernode; a range over the supernode's capacity, reachable only with
// duplicate ids, which are flagged, is emptied), then the level's list of the
// kind's tasks: one entry (supernode, tile row << 16 | tile column) per tile
// that has work, in supernode order, and the list's length (2 x length + 1 if
// its tiles are the small ones).  The products launch one workgroup per entry
// of the list's capacity; those past its length return after one uniform load
// (a grid laid out by supernode and static column capacity would have most of
// its workgroups find no columns, each after three dependent loads).  8, 13 and
// 15 us for 200, 1000 and 3000 contacts; 13, 19 and 30 with a workgroup for all
// kinds of a level.
constexpr int PLAN_NT = 1024;     // threads
constexpr int PLAN_CHUNK = 256;   // supernodes per chunk (levels with more take several)
constexpr int PLAN_KEYS = 4096;
__global__ __launch_bounds__(PLAN_NT) void k_rhs_plan(int nc, const int *__restrict__ level_first,
                                                      const int *__restrict__ level_sup,
                                                      const SupDev *__restrict__ sup, const int *__restrict__ keys,
                                                      int *__restrict__ lohi, const int *__restrict__ task_off,
                                                      int *__restrict__ task_cnt, int2 *__restrict__ tasks) {
  __shared__ int pre[PLAN_CHUNK];
  __shared__ int wsum[PLAN_CHUNK / 64];
  __shared__ int wtot;
  __shared__ int ssup[PLAN_CHUNK], sr[PLAN_CHUNK], snt[PLAN_CHUNK];
  __shared__ int skeys[PLAN_KEYS];
  const int l = blockIdx.x, k = blockIdx.y, tid = threadIdx.x, ln = tid & 63, wv = tid >> 6;
  const int first = level_first[l], last = level_first[l + 1];
  // the sorted keys are searched in LDS when they fit
  const int *kp = keys;
  if (nc <= PLAN_KEYS) {
    for (int i = tid; i < nc; i += PLAN_NT) skeys[i] = keys[i];
    kp = skeys;
  }
  if (tid == 0) wtot = 0;
  __syncthreads();
  // the kind's number of tiles of 64 (the workgroup of kind 0 stores the ranges)
  auto range = [&](const SupDev &S, int sn, int &lo, int &own, int &hi) {
    lo = lower_bound_i(kp, nc, S.first_desc);
    own = lower_bound_i(kp, nc, sn);
    hi = lower_bound_i(kp, nc, sn + 1);
    if (3 * (hi - lo) > S.rmax) own = hi = lo;
  };
  for (int q = first + tid; q < last; q += PLAN_NT) {
    const int sn = level_sup[q];
    const SupDev &S = sup[sn];
    int lo, own, hi;
    range(S, sn, lo, own, hi);
    if (k == 0) {
      lohi[3 * sn + 0] = lo;
      lohi[3 * sn + 1] = own;
      lohi[3 * sn + 2] = hi;
    }
    const int c = rhs_task_count(k, 3 * (hi - lo), 3 * S.ncol, 3 * S.nb, RHS_T);
    if (c) atomicAdd(&wtot, c);
  }
  __syncthreads();
  const int T = k != RT_ASM && wtot < RHS_SMALL ? RHS_TS : RHS_T;
  __syncthreads();
  int run = 0;
  for (int base = first; base < last; base += PLAN_CHUNK) {
    // task counts and their exclusive prefix over the chunk (waves
    // 0 .. PLAN_CHUNK / 64 - 1)
    const int q = base + tid;
    int c = 0, v = 0;
    if (tid < PLAN_CHUNK) {
      if (q < last) {
        const int sn = level_sup[q];
        const SupDev &S = sup[sn];
        int lo, own, hi;
        range(S, sn, lo, own, hi);
        const int r = 3 * (hi - lo), n3 = 3 * S.ncol, b3 = 3 * S.nb;
        c = rhs_task_count(k, r, n3, b3, T);
        ssup[tid] = sn;
        sr[tid] = (r + T - 1) / T;
        snt[tid] = ((k == RT_DIAG ? n3 : b3) + T - 1) / T;
      }
      v = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, 64);
        if (ln >= o) v += t;
      }
      if (ln == 63) wsum[wv] = v;
    }
    __syncthreads();
    if (tid == 0) {
      int acc = 0;
      for (int w = 0; w < PLAN_CHUNK / 64; ++w) {
        const int t = wsum[w];
        wsum[w] = acc;
        acc += t;
      }
      wtot = acc;
    }
    __syncthreads();
    if (tid < PLAN_CHUNK) pre[tid] = wsum[wv] + v - c;
    __syncthreads();
    // the chunk's tasks, all threads
    const int nq = min(PLAN_CHUNK, last - base), tot = wtot;
    int2 *out = tasks + task_off[RHS_KINDS * l + k] + run;
    for (int t = tid; t < tot; t += PLAN_NT) {
      int a = 0, b = nq;   // first q with pre > t; the task's supernode is the one before
      while (a < b) {
        const int mid = (a + b) >> 1;
        if (pre[mid] <= t)
          a = mid + 1;
        else
          b = mid;
      }
      const int qq = a - 1, u = t - pre[qq];
      int ti = u, tj = 0;
      if (k != RT_ASM) band_index(u, snt[qq], sr[qq], ti, tj);
      if (k == RT_DIAG) ti = snt[qq] - 1 - ti;   // deepest row tiles first (their product runs over k < i0 + T)
      out[t] = make_int2(ssup[qq], (ti << 16) | tj);
    }
    run += tot;
    __syncthreads();
  }
  if (tid == 0) task_cnt[RHS_KINDS * l + k] = 2 * run + (T == RHS_TS ? 1 : 0);
}

// ---- multi-RHS forward ------------------------------------------------------

// What the children's updates leave open of X_s, column by column (one wave
// per column, 4 columns per task): a column of an own contact is a unit vector
// of H^T (or a column of J^T = H^T C^T when frames are given); a column of a
// contact below a child is zero on the front rows that the child does not
// reach, the others are stored by the child's product.  With a residual R (the
// correction solve of the refinement) every column holds R_s on the
// supernode's own rows and zero below, and the children's products add to it.
// Everything that identifies the column is uniform over the wave.
template <class E>
__device__ inline void rhs_init_column(const SupDev *__restrict__ sup, int s, int jc, int l,
                                       const int *__restrict__ child, const int *__restrict__ invmap_off,
                                       const int *__restrict__ invmap, const int *__restrict__ lohi,
                                       const int *__restrict__ order, const int *__restrict__ node_ids,
                                       const int *__restrict__ iperm, const double *__restrict__ frames,
                                       const double *__restrict__ R, E *__restrict__ X) {
  const SupDev S = sup[s];
  const int lo = lohi[3 * s], own = lohi[3 * s + 1], hi = lohi[3 * s + 2];
  const int r = 3 * (hi - lo);
  if (jc >= r) return;
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  E *Xc = X + S.x_off + (long)jc * f;
  const int p = lo + jc / 3, a = jc % 3;
  if (R) {
    const double *Rc = R + S.z_off + (long)jc * n3;
    for (int i = l; i < f; i += 64) Xc[i] = (i < n3) ? E(Rc[i]) : E(0);
    return;
  }
  if (p >= own) {
    const int c = order[p];
    const int base = 3 * (iperm[node_ids[c]] - S.col0);
    for (int i = l; i < f; i += 64) {
      double v;
      if (frames == nullptr)
        v = (i == base + a) ? 1.0 : 0.0;
      else
        v = (i >= base && i < base + 3) ? frames[9L * c + 3 * a + (i - base)] : 0.0;
      Xc[i] = E(v);
    }
    return;
  }
  const int *im = nullptr;   // null: not below any child (cannot happen for sorted contacts)
  for (int q = 0; q < S.nchild; ++q) {
    const int ch = child[S.child_off + q];
    if (p >= lohi[3 * ch] && p < lohi[3 * ch + 2]) {
      if (sup[ch].nb == S.ncol + S.nb) return;   // the child reaches every row
      im = invmap + invmap_off[S.child_off + q];
      break;
    }
  }
  for (int i = l; i < S.ncol + S.nb; i += 64)
    if (im == nullptr || im[i] < 0)
      for (int a_ = 0; a_ < 3; ++a_) Xc[3 * i + a_] = E(0);
}

// All levels in one launch: asm_first[l] is the first workgroup of level l.
template <class E>
__global__ __launch_bounds__(256) void k_rhs_init(const SupDev *__restrict__ sup, int nlev,
                                                  const int *__restrict__ asm_first, const int *__restrict__ task_off,
                                                  const int *__restrict__ task_cnt, const int2 *__restrict__ tasks,
                                                  const int *__restrict__ child, const int *__restrict__ invmap_off,
                                                  const int *__restrict__ invmap, const int *__restrict__ lohi,
                                                  const int *__restrict__ order, const int *__restrict__ node_ids,
                                                  const int *__restrict__ iperm, const double *__restrict__ frames,
                                                  const double *__restrict__ R, E *__restrict__ X) {
  int l = 0;
  while (l + 1 < nlev && asm_first[l + 1] <= (int)blockIdx.x) ++l;
  const int t = blockIdx.x - asm_first[l];
  if (t >= task_cnt[RHS_KINDS * l + RT_ASM] >> 1) return;
  const int2 tk = tasks[task_off[RHS_KINDS * l + RT_ASM] + t];
  rhs_init_column<E>(sup, tk.x, 4 * (tk.y >> 16) + (threadIdx.x >> 6), threadIdx.x & 63, child, invmap_off, invmap,
                     lohi, order, node_ids, iperm, frames, R, X);
}

// The product kernels' tiles hold the transposed product (the accumulator's
// columns are the rows of the column-major output), so that 16 lanes store 16
// neighbours.  W_H of 200 contacts at 9 450 DOF: 497 -> 345 us, of 1000 at
// 61 236: 2.65 -> 2.10 ms, of 3000 at 75 600: 11.8 -> 9.7 ms.
template <class E>
struct RhsAcc {
  typedef AccMT<2, 32, E> Mid;     // 64 x 64, K-chunk 32
  typedef AccMT<1, 64, E> Small;   // 32 x 32, K-chunk 64
  static constexpr int LDS = Mid::LDS > Small::LDS ? Mid::LDS : Small::LDS;
  static_assert(Mid::T == RHS_T && Small::T == RHS_TS, "tile edges of the plan");
};

// Task of this workgroup (false: none); small: it is a 32 x 32 tile.
__device__ inline bool rhs_my_task(const int2 *__restrict__ tasks, const int *__restrict__ ntask, int2 &tk,
                                   bool &small) {
  const int n = *ntask;
  if ((int)blockIdx.x >= n >> 1) return false;
  tk = tasks[blockIdx.x];
  small = n & 1;
  return true;
}

// Z_s = L_ss^{-1} X_s[:n_s], one tile per task.  z64 (FP32 solves of
// the mixed-precision build): 1 also stores the tile into the FP64 Z,
// 2 adds it there (a refinement correction).
template <class Ac>
__device__ void rhs_diag_tile(const SupDev &S, int r, int2 tk, const typename Ac::elem *__restrict__ linv,
                              const typename Ac::elem *__restrict__ X, typename Ac::elem *__restrict__ Z,
                              double *__restrict__ Z64, int z64, typename Ac::elem *lds) {
  typedef typename Ac::elem E;
  constexpr int T = Ac::T;
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  const int i0 = T * (tk.y >> 16), j0 = T * (tk.y & 0xffff);
  if (i0 >= n3 || j0 >= r) return;
  const int M = min(T, n3 - i0), N = min(T, r - j0);
  const int kend = min(n3, i0 + T);
  Ac acc;
  acc.zero();
  acc.template acc<false, true>(X + S.x_off + (long)j0 * f, f, linv + S.linv_off + i0, n3, N, M, 0, kend, lds);
  const long out = S.z_off + i0 + (long)j0 * n3;
  acc.put(Z + out, n3, N, M, [](E v) { return v; });
  if (z64 == 1) acc.put(Z64 + out, n3, N, M, [](E v) { return (double)v; });
  if (z64 == 2)
    acc.update(Z64 + out, n3, Z64 + out, n3, N, M, [](int, int) { return true; },
               [](int, int, E v, double old) { return old + (double)v; });
}
template <class E>
__global__ __launch_bounds__(256) void k_rhs_diag(const SupDev *__restrict__ sup, const int2 *__restrict__ tasks,
                                                  const int *__restrict__ ntask, const int *__restrict__ lohi,
                                                  const E *__restrict__ linv, const E *__restrict__ X,
                                                  E *__restrict__ Z, double *__restrict__ Z64, int z64) {
  __shared__ E lds[RhsAcc<E>::LDS];
  int2 tk;
  bool small;
  if (!rhs_my_task(tasks, ntask, tk, small)) return;
  const int s = tk.x;
  const SupDev S = sup[s];
  const int r = 3 * (lohi[3 * s + 2] - lohi[3 * s]);
  if (small)
    rhs_diag_tile<typename RhsAcc<E>::Small>(S, r, tk, linv, X, Z, Z64, z64, lds);
  else
    rhs_diag_tile<typename RhsAcc<E>::Mid>(S, r, tk, linv, X, Z, Z64, z64, lds);
}

// X_parent = X_s[n_s:] - L_21 Z_s on the front rows below s, one tile per
// task; added there when the parents' columns hold a residual.  The store goes
// straight to the parent's front, in place of a store to X_s and a kernel per
// level that gathered the children's rows (8 to 24 us a level at 200 to 1000
// contacts, and three passes over X).  W_H of 1000 contacts at 61 236 DOF:
// 2.10 -> 1.97 ms, of 400 mapped ones at 12 288: 475 -> 426 us.
template <class Ac>
__device__ void rhs_off_tile(const SupDev &S, int r, int2 tk, const typename Ac::elem *__restrict__ front,
                             const typename Ac::elem *__restrict__ Z, const typename Ac::elem *__restrict__ X,
                             const int *__restrict__ rel, typename Ac::elem *__restrict__ Xp, long fp, bool add,
                             typename Ac::elem *lds) {
  constexpr int T = Ac::T;
  const int n3 = 3 * S.ncol, b3 = 3 * S.nb, f = n3 + b3;
  const int i0 = T * (tk.y >> 16), j0 = T * (tk.y & 0xffff);
  if (i0 >= b3 || j0 >= r) return;
  const int M = min(T, b3 - i0), N = min(T, r - j0);
  Ac acc;
  acc.zero();
  acc.template acc<false, true>(Z + S.z_off + (long)j0 * n3, n3, front + S.front_off + n3 + i0, f, N, M, 0, n3, lds);
  acc.push(Xp + (long)j0 * fp, fp, [&](int i) { return 3 * rel[(i0 + i) / 3] + (i0 + i) % 3; },
           X + S.x_off + n3 + i0 + (long)j0 * f, f, N, M, add);
}
template <class E>
__global__ __launch_bounds__(256) void k_rhs_off(const SupDev *__restrict__ sup, const int2 *__restrict__ tasks,
                                                 const int *__restrict__ ntask, const int *__restrict__ lohi,
                                                 const int *__restrict__ relmap, const E *__restrict__ front,
                                                 const E *__restrict__ Z, E *X, int add) {
  __shared__ E lds[RhsAcc<E>::LDS];
  int2 tk;
  bool small;
  if (!rhs_my_task(tasks, ntask, tk, small)) return;
  const int s = tk.x;
  const SupDev S = sup[s];
  const int lo = lohi[3 * s], hi = lohi[3 * s + 2], r = 3 * (hi - lo);
  // the parent's columns of these contacts; none if the plan emptied its range
  const int p = S.parent, plo = lohi[3 * p];
  if (lo < plo || hi > lohi[3 * p + 1]) return;
  const long fp = 3L * (sup[p].ncol + sup[p].nb);
  E *Xp = X + sup[p].x_off + 3L * (lo - plo) * fp;
  if (small)
    rhs_off_tile<typename RhsAcc<E>::Small>(S, r, tk, front, Z, X, relmap + S.rows_off, Xp, fp, add, lds);
  else
    rhs_off_tile<typename RhsAcc<E>::Mid>(S, r, tk, front, Z, X, relmap + S.rows_off, Xp, fp, add, lds);
}

// Residual of the forward solve on a supernode's own rows (FP64, the
// refinement of the mixed-precision build): R_s = X_s[:n_s] - L_ss Z_s with
// X_s in FP64, from the unit columns and the children's FP64
// updates; L_ss is the lower triangle of the front's diagonal block.
template <class Ac>
__device__ void rhs_resid_tile(const SupDev &S, int r, int2 tk, const double *__restrict__ front,
                               const double *__restrict__ X, const double *__restrict__ Z, double *__restrict__ R,
                               double *lds) {
  constexpr int T = Ac::T;
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  const int i0 = T * (tk.y >> 16), j0 = T * (tk.y & 0xffff);
  if (i0 >= n3 || j0 >= r) return;
  const int M = min(T, n3 - i0), N = min(T, r - j0);
  const int kend = min(n3, i0 + T);
  Ac acc;
  acc.zero();
  // B(k, i) = L_ss(i0 + i, k), zero above the diagonal (k > i0 + i)
  acc.template acc<false, true, true>(Z + S.z_off + (long)j0 * n3, n3, front + S.front_off + i0, f, N, M, 0, kend, lds,
                                      i0);
  acc.update(R + S.z_off + i0 + (long)j0 * n3, n3, X + S.x_off + i0 + (long)j0 * f, f, N, M,
             [](int, int) { return true; }, [](int, int, double v, double x) { return x - v; });
}
__global__ __launch_bounds__(256) void k_rhs_resid(const SupDev *__restrict__ sup, const int2 *__restrict__ tasks,
                                                   const int *__restrict__ ntask, const int *__restrict__ lohi,
                                                   const double *__restrict__ front, const double *__restrict__ X,
                                                   const double *__restrict__ Z, double *__restrict__ R) {
  __shared__ double lds[RhsAcc<double>::LDS];
  int2 tk;
  bool small;
  if (!rhs_my_task(tasks, ntask, tk, small)) return;
  const int s = tk.x;
  const SupDev S = sup[s];
  const int r = 3 * (lohi[3 * s + 2] - lohi[3 * s]);
  if (small)
    rhs_resid_tile<RhsAcc<double>::Small>(S, r, tk, front, X, Z, R, lds);
  else
    rhs_resid_tile<RhsAcc<double>::Mid>(S, r, tk, front, X, Z, R, lds);
}

__global__ void k_fill(long n, double v, double *__restrict__ x) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) x[i] = v;
}

// Wp = Z^T Z in supernode order of the contacts, one tile (I >= J) and its
// mirror image per workgroup.  Entry (i, j) sums over the supernodes above both
// contacts, which are the common part of their paths to the root: a tile below
// the diagonal meets the supernodes that hold its last column's and its first
// row's contact, one path; a diagonal tile meets the paths of all of its
// contacts (each supernode is taken at its first contact in the tile).  One
// launch after the solve, in place of one per level that added into Wp beside
// it on a second stream: the waits between the streams cost 10 us a level, and
// Wp was cleared, read and written once per level and mirrored.  W_H of 200
// contacts at 9 450 DOF: 303 -> 237 us, of 3000 at 75 600: 10.1 -> 9.5 to
// 10.0 ms; of 1000 at 61 236 it costs what it saves (2.04 -> 2.03 to 2.07 ms).
//
// Tile order: few tiles go by their distance from the diagonal, the longest
// paths first, WP_BAND or more in bands that share panels.  The two meet at
// about 2300 tiles where the paths are long (28 x 27 x 27 nodes, by distance and
// in bands: 1653 tiles 2.52 and 2.61 ms, 3655 tiles 4.36 and 4.10, 5886 tiles
// 6.24 and 5.66, 10 011 tiles 9.69 and 8.40) and at about 4096 where they are
// short (60 x 60 x 3 nodes: 2556 tiles 0.87 and 0.92, 4095 tiles 1.17 and 1.17,
// 5886 tiles 1.59 and 1.49; 12 x 12 x 80 nodes alike): the line is the one that
// costs neither.  Below WP_SMALL tiles of 64 the tiles are 32 x 32: at 1128
// tiles those cost 3 %.
constexpr int WP_SMALL = 512, WP_BAND = 4096;
struct WpSeg {
  long z;             // Z_s
  int n3, lo, hi;     // rows, contact range in DOF columns
};
template <class Ac>
__global__ __launch_bounds__(256) void k_wp_tiles(int nc, int nsup, bool band, const SupDev *__restrict__ sup,
                                                  const int *__restrict__ keys, const int *__restrict__ lohi,
                                                  const int *__restrict__ anc_ptr, const int *__restrict__ anc,
                                                  const double *__restrict__ Z, double *__restrict__ Wp) {
  constexpr int T = Ac::T;
  __shared__ double lds[Ac::LDS];
  __shared__ WpSeg seg[256];
  __shared__ int wcnt[4];
  static_assert(T * (T + 1) <= Ac::LDS, "the tile is turned in the staging space");
  const int m = 3 * nc, nt = (m + T - 1) / T;
  int I = blockIdx.x, J = I;
  if (band) {
    if (I >= nt) {
      band_tri_index(I - nt, nt - 1, I, J);
      ++I;
    }
  } else {
    tri_index(nt * (nt + 1) / 2 - 1 - blockIdx.x, I, J);
    I = J + nt - 1 - I;
  }
  const int i0 = T * I, j0 = T * J, M = min(T, m - i0), N = min(T, m - j0);
  const int tid = threadIdx.x, ln = tid & 63;
  const int p0 = i0 / 3, pc = (j0 + N - 1) / 3;            // first row's, last column's contact
  const int pend = I == J ? (i0 + M - 1) / 3 : p0;         // contacts whose paths are met
  Ac acc;
  acc.zero();
  // 16 contacts and 16 supernodes of each one's path at a time, from the root
  // down (one wave walked the contacts one after the other, dependent loads
  // each time: 54 against 50 us for Z^T Z of 200 contacts, 677 against 653 of
  // 1000)
  for (int pb = p0, db = 0; pb <= pend;) {
    const int p = pb + tid / 16;
    bool take = false, more = false;
    WpSeg sg = {};
    if (p <= pend) {
      const int own = keys[p];
      const int a0 = own < nsup ? anc_ptr[own] : 0, len = own < nsup ? anc_ptr[own + 1] - a0 : 0;
      const int d = len - 1 - db - tid % 16;
      more = len > db + 16;
      if (d >= 0) {
        const int s = anc[a0 + d], lo = lohi[3 * s], hi = lohi[3 * s + 2];
        take = hi > p && (I == J ? max(lo, p0) == p : lo <= pc);
        sg = {sup[s].z_off, 3 * sup[s].ncol, 3 * lo, 3 * hi};
      }
    }
    const unsigned long long mask = __ballot(take);
    if (ln == 0) wcnt[tid / 64] = __popcll(mask);
    more = __syncthreads_or(more);
    int at = __popcll(mask & ((1ull << ln) - 1)), nseg = 0;
    for (int w = 0; w < 4; ++w) {
      at += w < tid / 64 ? wcnt[w] : 0;
      nseg += wcnt[w];
    }
    if (take) seg[at] = sg;
    __syncthreads();
    nseg = __builtin_amdgcn_readfirstlane(nseg);
    if (more) {
      db += 16;
    } else {
      db = 0;
      pb += 16;
    }
    // their rows, chunk by chunk, the next chunk in flight
    if (nseg > 0)
      acc.chain_product(nseg, [&](int q, const double *&A, int &an, int &as, const double *&B, int &bn, int &bs, int &n3) {
        const WpSeg g = seg[q];
        n3 = __builtin_amdgcn_readfirstlane(g.n3);
        const int lo = __builtin_amdgcn_readfirstlane(g.lo), hi = __builtin_amdgcn_readfirstlane(g.hi);
        const long z = ((long)__builtin_amdgcn_readfirstlane((int)(g.z >> 32)) << 32) |
                       (unsigned)__builtin_amdgcn_readfirstlane((int)g.z);
        as = max(0, lo - i0);
        an = min(M, hi - i0) - as;
        bs = max(0, lo - j0);
        bn = min(N, hi - j0) - bs;
        A = Z + z + (long)(i0 + as - lo) * n3;
        B = Z + z + (long)(j0 + bs - lo) * n3;
      }, lds);
  }
  // the lower part from the tile, the upper part turned
  __syncthreads();
  acc.for_each([&](int i, int j, double v) { lds[i * (T + 1) + j] = v; });
  __syncthreads();
  for (int e = tid; e < T * T; e += 256) {
    const int i = e / T, j = e % T;
    if (i < M && j < N) Wp[(long)(i0 + i) * m + j0 + j] = I == J && j > i ? lds[j * (T + 1) + i] : lds[i * (T + 1) + j];
  }
  if (I != J)
    for (int e = tid; e < T * T; e += 256) {
      const int j = e / T, i = e % T;
      if (i < M && j < N) Wp[(long)(j0 + j) * m + i0 + i] = lds[i * (T + 1) + j];
    }
}

// W_H[3c+a][3c'+b] = Wp[3 pos(c) + a][3 pos(c') + b] (Wp symmetric): one
// block per output row, the source row stays in cache.
template <class TW>
__global__ __launch_bounds__(256) void k_wh_unpermute(int nc, const int *__restrict__ pos, const double *__restrict__ Wp,
                                                      TW *__restrict__ WH) {
  const int m = 3 * nc;
  const int i = blockIdx.x;
  const double *src = Wp + (long)(3 * pos[i / 3] + i % 3) * m;
  TW *dst = WH + (long)i * m;
  for (int j = threadIdx.x; j < m; j += 256) dst[j] = (TW)src[3 * pos[j / 3] + j % 3];
}

__global__ void k_to_float(long n, const double *__restrict__ x, float *__restrict__ y) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (float)x[i];
}

__global__ void k_to_double(long n, const float *__restrict__ x, double *__restrict__ y) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (double)x[i];
}

// Mapped contacts (Eq. 6): contact a is the point sum_k w_ak x(u_ak) over up
// to four slots (unused slots: index -1), so H = Hw Hn with Hn the nodal
// selection of the distinct nodes and
//   W_H[3a+i][3b+j] = sum_{k,l} w_ak w_bl W_N[3 u_ak + i][3 u_bl + j],
// W_N = Hn A^-1 Hn^T (built by the nodal path).  A thread has one column
// 3b + j of contact row a (blockIdx.y), so that three lanes read the three
// neighbouring doubles of a block's row and 64 lanes store neighbours; its 48
// loads are in flight together.  The sixteen terms are summed in an order that
// is the same for (a, b) and (b, a) -- diagonal slot pairs, then each
// off-diagonal pair (k, l) as t_kl + t_lk -- with products and sums rounded
// separately (no contraction), so W_H is exactly symmetric like W_N.
// 70 -> 45 us for 400 contacts over 502 nodes, 9.5 -> 2.5 ms for 3000 contacts
// of two bodies (a thread per block: three times the cache lines a load).
__global__ __launch_bounds__(256) void k_wh_expand(int nc, int nu3, const int *__restrict__ idx,
                                                   const double *__restrict__ wts, const double *__restrict__ WN,
                                                   double *__restrict__ WH) {
  const int a = blockIdx.y, e = 256 * blockIdx.x + threadIdx.x;
  const long m = 3L * nc;
  if (e >= m) return;
  const int b = e / 3, j = e % 3;
  int ua[4], ub[4];
  double wa[4], wb[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ua[k] = idx[4 * a + k];
    wa[k] = ua[k] >= 0 ? wts[4 * a + k] : 0.0;
    ub[k] = idx[4 * b + k];
    wb[k] = ub[k] >= 0 ? wts[4 * b + k] : 0.0;
  }
  // t(k, l)[i] = (w_ak w_bl) W_N[3 u_ak + i][3 u_bl + j], 0 for an unused slot
  double t[4][4][3];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      const bool used = ua[k] >= 0 && ub[l] >= 0;
      const double *x = WN + (long)(3 * max(ua[k], 0)) * nu3 + 3 * max(ub[l], 0) + j;
#pragma unroll
      for (int i = 0; i < 3; ++i) t[k][l][i] = used ? x[(long)i * nu3] : 0.0;
    }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    auto term = [&](int k, int l) -> double {
      return ua[k] >= 0 && ub[l] >= 0 ? __dmul_rn(__dmul_rn(wa[k], wb[l]), t[k][l][i]) : 0.0;
    };
    double acc = term(0, 0);
#pragma unroll
    for (int k = 1; k < 4; ++k) acc = __dadd_rn(acc, term(k, k));
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int l = k + 1; l < 4; ++l) acc = __dadd_rn(acc, __dadd_rn(term(k, l), term(l, k)));
    WH[(3L * a + i) * m + e] = acc;
  }
}

// ---- single RHS -------------------------------------------------------------

// Single-RHS products, 1024 threads per block.  Column-major A times x: lane
// = row (64 rows, coalesced), wave = k-phase (16 phases), four independent
// accumulators per thread, phases summed in a fixed order through LDS.
// Transposed products: one wave per column, 16 columns per block, the
// vector staged in LDS once per block.
constexpr int GV_R = 64, GV_P = 16, GV_X = 4096;
constexpr int ZF_K = 256;   // columns of Z per chunk of the Z f product

__device__ inline double gemv_part(const double *__restrict__ A, long lda, const double *__restrict__ x, int i,
                                   int nrows, int k0, int k1, int ph) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  if (i < nrows) {
    int k = k0 + ph;
    for (; k + 3 * GV_P < k1; k += 4 * GV_P) {
      a0 = fma(A[i + (long)k * lda], x[k], a0);
      a1 = fma(A[i + (long)(k + GV_P) * lda], x[k + GV_P], a1);
      a2 = fma(A[i + (long)(k + 2 * GV_P) * lda], x[k + 2 * GV_P], a2);
      a3 = fma(A[i + (long)(k + 3 * GV_P) * lda], x[k + 3 * GV_P], a3);
    }
    for (; k < k1; k += GV_P) a0 = fma(A[i + (long)k * lda], x[k], a0);
  }
  return (a0 + a1) + (a2 + a3);
}

// Sum of the 16 phase partials of row r (valid in wave 0).
__device__ inline double phase_sum(double v, double (*part)[GV_R + 1]) {
  const int r = threadIdx.x & 63, ph = threadIdx.x >> 6;
  part[ph][r] = v;
  __syncthreads();
  double t = 0.0;
  if (ph == 0)
    for (int q = 0; q < GV_P; ++q) t += part[q][r];
  return t;
}

// Entry i of the single-RHS front of supernode S (Eq. 12 forward half): the
// permuted right-hand side on its own columns plus the children's update
// entries mapped onto row i (extend-add), children in order.
__device__ inline double fwd1_front(const SupDev &S, int i, const SupDev *__restrict__ sup,
                                    const int *__restrict__ child, const int *__restrict__ invmap_off,
                                    const int *__restrict__ invmap, const int *__restrict__ perm,
                                    const double *__restrict__ b, const double *__restrict__ x1) {
  const int n3 = 3 * S.ncol;
  double v = (i < n3) ? b[3 * perm[S.col0 + i / 3] + i % 3] : 0.0;
  for (int c = 0; c < S.nchild; ++c) {
    const int ii = invmap[invmap_off[S.child_off + c] + i / 3];
    if (ii >= 0) {
      const SupDev C = sup[child[S.child_off + c]];
      v += x1[C.x1_off + 3 * C.ncol + 3 * ii + i % 3];
    }
  }
  return v;
}

// The single-RHS products take block x from a static task list of their
// level: (supernode of the level, block of 64 rows or 16 columns), only the
// blocks a supernode has.  Split-K (top tree levels, where a level has too
// few row blocks to fill the GPU): block y = chunk of k; each block writes
// the sums over its chunk to part[(task * nsplit + chunk) * 64 + row] and
// k_fwd1_fin adds the nsplit partials in chunk order.  nsplit = 1: the row
// block's sums are final.  Returns true when they are (wave 0: row sums).
__device__ inline bool fwd1_split_store(double t, double *__restrict__ part) {
  const int nsplit = gridDim.y;
  if (nsplit == 1) return true;
  const int r = threadIdx.x & 63, ph = threadIdx.x >> 6;
  if (ph == 0) part[((long)blockIdx.x * nsplit + blockIdx.y) * GV_R + r] = t;
  return false;
}

// Chunk [ka, kb) of k in [0, kend) for chunk ks of nsplit (multiples of GV_P).
__device__ inline void fwd1_chunk(int kend, int nsplit, int ks, int &ka, int &kb) {
  const int kc = ((kend + nsplit - 1) / nsplit + GV_P - 1) / GV_P * GV_P;
  ka = min(kend, ks * kc);
  kb = min(kend, ka + kc);
}

// y[3 col0 + i] = sum_{k <= i} Linv(i, k) x1_s[k]; the front entries it needs
// are assembled on the fly into LDS (GV_X at a time)
__global__ __launch_bounds__(1024) void k_fwd1_diag(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                    const int2 *__restrict__ tasks, const int *__restrict__ child,
                                                    const int *__restrict__ invmap_off, const int *__restrict__ invmap,
                                                    const int *__restrict__ perm, const double *__restrict__ b,
                                                    const double *__restrict__ linv, const double *__restrict__ x1,
                                                    double *__restrict__ y, double *__restrict__ part) {
  __shared__ double ps[GV_P][GV_R + 1];
  __shared__ double xs[GV_X];
  const int2 tk = tasks[blockIdx.x];
  const SupDev S = sup[level_sup[tk.x]];
  const int n3 = 3 * S.ncol;
  const int i0 = GV_R * tk.y;
  const int r = threadIdx.x & 63, ph = threadIdx.x >> 6, i = i0 + r;
  const int kend = min(n3, i0 + GV_R);
  int ka, kb;
  fwd1_chunk(kend, gridDim.y, blockIdx.y, ka, kb);
  double v = 0.0;
  for (int kk = ka; kk < kb; kk += GV_X) {
    const int kn = min(kb, kk + GV_X);
    __syncthreads();
    for (int k = kk + threadIdx.x; k < kn; k += 1024)
      xs[k - kk] = fwd1_front(S, k, sup, child, invmap_off, invmap, perm, b, x1);
    __syncthreads();
    v += gemv_part(linv + S.linv_off, n3, xs - kk, i, n3, kk, kn, ph);
  }
  const double t = phase_sum(v, ps);
  if (!fwd1_split_store(t, part)) return;
  if (ph == 0 && i < n3) y[3 * S.col0 + i] = t;
}

// x1_s[n_s + i] = front(n_s + i) - sum_k L21(i, k) y_s[k]
__global__ __launch_bounds__(1024) void k_fwd1_off(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                   const int2 *__restrict__ tasks, const int *__restrict__ child,
                                                   const int *__restrict__ invmap_off,
                                                   const int *__restrict__ invmap, const int *__restrict__ perm,
                                                   const double *__restrict__ b, const double *__restrict__ front,
                                                   const double *__restrict__ y, double *__restrict__ x1,
                                                   double *__restrict__ part) {
  __shared__ double ps[GV_P][GV_R + 1];
  const int2 tk = tasks[blockIdx.x];
  const SupDev S = sup[level_sup[tk.x]];
  const int n3 = 3 * S.ncol, b3 = 3 * S.nb, f = n3 + b3;
  const int i0 = GV_R * tk.y;
  const int r = threadIdx.x & 63, ph = threadIdx.x >> 6, i = i0 + r;
  int ka, kb;
  fwd1_chunk(n3, gridDim.y, blockIdx.y, ka, kb);
  const double v = gemv_part(front + S.front_off + n3, f, y + 3 * S.col0, i, b3, ka, kb, ph);
  const double t = phase_sum(v, ps);
  if (!fwd1_split_store(t, part)) return;
  if (ph == 0 && i < b3)
    x1[S.x1_off + n3 + i] = fwd1_front(S, n3 + i, sup, child, invmap_off, invmap, perm, b, x1) - t;
}

// The sums of split products (one wave per row block): off = 0 writes y of
// the diagonal product, off = 1 the below rows of x1.
__global__ __launch_bounds__(64) void k_fwd1_fin(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                 const int2 *__restrict__ tasks, const int *__restrict__ child,
                                                 const int *__restrict__ invmap_off,
                                                 const int *__restrict__ invmap, const int *__restrict__ perm,
                                                 const double *__restrict__ b, int off, int nsplit,
                                                 const double *__restrict__ part, double *__restrict__ y,
                                                 double *__restrict__ x1) {
  const int2 tk = tasks[blockIdx.x];
  const SupDev S = sup[level_sup[tk.x]];
  const int n3 = 3 * S.ncol, rows = off ? 3 * S.nb : n3;
  const int i = GV_R * tk.y + (int)threadIdx.x;
  if (i >= rows) return;
  double t = 0.0;
  for (int q = 0; q < nsplit; ++q) t += part[((long)blockIdx.x * nsplit + q) * GV_R + threadIdx.x];
  if (off)
    x1[S.x1_off + n3 + i] = fwd1_front(S, n3 + i, sup, child, invmap_off, invmap, perm, b, x1) - t;
  else
    y[3 * S.col0 + i] = t;
}

// y_s[j] -= sum_i L21(i, j) x[below row i]
__global__ __launch_bounds__(1024) void k_bwd1_off(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                   const int2 *__restrict__ tasks, const int *__restrict__ rows,
                                                   const double *__restrict__ front, const double *__restrict__ xp,
                                                   double *__restrict__ y) {
  __shared__ double xg[GV_X];
  const int2 tk = tasks[blockIdx.x];
  const SupDev S = sup[level_sup[tk.x]];
  const int n3 = 3 * S.ncol, b3 = 3 * S.nb, f = n3 + b3;
  const int j0 = GV_P * tk.y;
  const int *rw = rows + S.rows_off;
  const int bs = min(b3, GV_X);
  for (int i = threadIdx.x; i < bs; i += 1024) xg[i] = xp[3 * rw[i / 3] + i % 3];
  __syncthreads();
  const int j = j0 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (j >= n3) return;
  const double *F = front + S.front_off + n3 + (long)j * f;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int i = l;
  for (; i + 192 < bs; i += 256) {
    a0 = fma(F[i], xg[i], a0);
    a1 = fma(F[i + 64], xg[i + 64], a1);
    a2 = fma(F[i + 128], xg[i + 128], a2);
    a3 = fma(F[i + 192], xg[i + 192], a3);
  }
  for (; i < bs; i += 64) a0 = fma(F[i], xg[i], a0);
  for (; i < b3; i += 64) a0 = fma(F[i], xp[3 * rw[i / 3] + i % 3], a0);
  double acc = (a0 + a1) + (a2 + a3);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (l == 0) y[3 * S.col0 + j] -= acc;
}

// xp[3 col0 + j] = sum_{i >= j} Linv(i, j) y_s[i]
__global__ __launch_bounds__(1024) void k_bwd1_diag(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                    const int2 *__restrict__ tasks, const double *__restrict__ linv,
                                                    const double *__restrict__ y, double *__restrict__ xp) {
  __shared__ double yg[GV_X];
  const int2 tk = tasks[blockIdx.x];
  const SupDev S = sup[level_sup[tk.x]];
  const int n3 = 3 * S.ncol;
  const int j0 = GV_P * tk.y;
  const double *ys = y + 3 * S.col0;
  const int ns = min(n3, GV_X);
  for (int i = j0 + threadIdx.x; i < ns; i += 1024) yg[i] = ys[i];
  __syncthreads();
  const int j = j0 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (j >= n3) return;
  const double *Lc = linv + S.linv_off + (long)j * n3;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int i = j + l;
  for (; i + 192 < ns; i += 256) {
    a0 = fma(Lc[i], yg[i], a0);
    a1 = fma(Lc[i + 64], yg[i + 64], a1);
    a2 = fma(Lc[i + 128], yg[i + 128], a2);
    a3 = fma(Lc[i + 192], yg[i + 192], a3);
  }
  for (; i < ns; i += 64) a0 = fma(Lc[i], yg[i], a0);
  for (; i < n3; i += 64) a0 = fma(Lc[i], ys[i], a0);
  double acc = (a0 + a1) + (a2 + a3);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (l == 0) xp[3 * S.col0 + j] = acc;
}

__global__ void k_unpermute_vec(int N, const int *__restrict__ perm, const double *__restrict__ xp,
                                double *__restrict__ x) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  int v = perm[p];
  x[3 * v] = xp[3 * p];
  x[3 * v + 1] = xp[3 * p + 1];
  x[3 * v + 2] = xp[3 * p + 2];
}

}  // namespace

namespace {

void backward_solve(icr_scene *s, double *x) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  const int nl = (int)F.levels.size();
  double *y = F.d_y, *xp = F.d_y + s->mesh.n;
  for (int l = nl - 1; l >= 0; --l) {
    const LevelInfo &L = F.levels[l];
    if (!L.count) continue;
    const int *ls = F.d_level_sup + L.first;
    const int2 *tb = F.d_srhs_tasks + L.srhs_off[SR_BWD];
    const unsigned nb = (unsigned)L.srhs_cnt[SR_BWD];
    if (L.max_b3 > 0) {
      k_bwd1_off<<<nb, 1024, 0, st>>>(F.d_sup, ls, tb, F.d_rows, F.d_front, xp, y);
      ICR_LAUNCH_CHECK();
    }
    k_bwd1_diag<<<nb, 1024, 0, st>>>(F.d_sup, ls, tb, F.d_linv, y, xp);
    ICR_LAUNCH_CHECK();
  }
  k_unpermute_vec<<<cdiv(s->mesh.N, 256), 256, 0, st>>>(s->mesh.N, F.d_perm, xp, x);
  ICR_LAUNCH_CHECK();
}

// y[3 col0_s + i] = sum_c Z_s(i, c) f[contact at column c]: the forward half of
// A^-1 H^T f reuses Z = L^-1 P H^T from the W_H build of the same contacts.
// k_zf_part: one task = 64 rows x one chunk of ZF_K columns of Z_s, partial
// sums to part[off + chunk n3 + row]; k_zf_sum adds the chunks in order.
__global__ __launch_bounds__(1024) void k_zf_part(const int4 *__restrict__ tasks, const SupDev *__restrict__ sup,
                                                  const int *__restrict__ lohi, const double *__restrict__ Z,
                                                  const double *__restrict__ fpos, double *__restrict__ part) {
  __shared__ double ps[GV_P][GV_R + 1];
  const int4 tk = tasks[blockIdx.x];
  const int s = tk.x, i0 = tk.y, k0 = tk.z;
  const SupDev S = sup[s];
  const int n3 = 3 * S.ncol;
  const int lo = lohi[3 * s], r = 3 * (lohi[3 * s + 2] - lo);
  if (k0 >= r && k0 > 0) return;   // chunk beyond this call's columns (chunk 0 always writes)
  const int rr = threadIdx.x & 63, ph = threadIdx.x >> 6, i = i0 + rr;
  const double v = gemv_part(Z + S.z_off, n3, fpos + 3 * lo, i, n3, k0, min(r, k0 + ZF_K), ph);
  const double t = phase_sum(v, ps);
  if (ph == 0 && i < n3) part[tk.w + (long)(k0 / ZF_K) * n3 + i] = t;
}
__global__ void k_zf_sum(const int4 *__restrict__ tasks, const SupDev *__restrict__ sup,
                         const int *__restrict__ lohi, const double *__restrict__ part, double *__restrict__ y) {
  const int4 tk = tasks[blockIdx.x];
  const int s = tk.x, i = tk.y + (int)threadIdx.x;
  const SupDev S = sup[s];
  const int n3 = 3 * S.ncol;
  if (i >= n3) return;
  const int r = 3 * (lohi[3 * s + 2] - lohi[3 * s]);
  const int nch = max(1, (r + ZF_K - 1) / ZF_K);
  double acc = 0.0;
  for (int ch = 0; ch < nch; ++ch) acc += part[tk.w + (long)ch * n3 + i];
  y[3 * S.col0 + i] = acc;
}

// fpos[3 p + a] = f[3 order[p] + a]
__global__ void k_gather_fpos(int nc, const int *__restrict__ order, const double *__restrict__ f,
                              double *__restrict__ fpos) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= 3 * nc) return;
  fpos[e] = f[3 * order[e / 3] + e % 3];
}

}  // namespace

void single_rhs_solve(icr_scene *s, const double *b, double *x) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  const int nl = (int)F.levels.size();
  double *y = F.d_y;
  for (int l = 0; l < nl; ++l) {
    const LevelInfo &L = F.levels[l];
    if (!L.count) continue;
    const int *ls = F.d_level_sup + L.first;
    const int2 *td = F.d_srhs_tasks + L.srhs_off[SR_FWD_DIAG], *to = F.d_srhs_tasks + L.srhs_off[SR_FWD_OFF];
    const unsigned nd = (unsigned)L.srhs_cnt[SR_FWD_DIAG], no = (unsigned)L.srhs_cnt[SR_FWD_OFF];
    k_fwd1_diag<<<dim3(nd, L.fwd_split_diag), 1024, 0, st>>>(F.d_sup, ls, td, F.d_child, F.d_invmap_off, F.d_invmap,
                                                              F.d_perm, b, F.d_linv, F.d_x1, y, F.d_fwd_part);
    ICR_LAUNCH_CHECK();
    if (L.fwd_split_diag > 1) {
      k_fwd1_fin<<<nd, 64, 0, st>>>(F.d_sup, ls, td, F.d_child, F.d_invmap_off, F.d_invmap, F.d_perm, b, 0,
                                    L.fwd_split_diag, F.d_fwd_part, y, F.d_x1);
      ICR_LAUNCH_CHECK();
    }
    if (no > 0) {
      k_fwd1_off<<<dim3(no, L.fwd_split_off), 1024, 0, st>>>(F.d_sup, ls, to, F.d_child, F.d_invmap_off, F.d_invmap,
                                                              F.d_perm, b, F.d_front, y, F.d_x1, F.d_fwd_part);
      ICR_LAUNCH_CHECK();
      if (L.fwd_split_off > 1) {
        k_fwd1_fin<<<no, 64, 0, st>>>(F.d_sup, ls, to, F.d_child, F.d_invmap_off, F.d_invmap, F.d_perm, b, 1,
                                      L.fwd_split_off, F.d_fwd_part, y, F.d_x1);
        ICR_LAUNCH_CHECK();
      }
    }
  }
  backward_solve(s, x);
}

void contact_force_solve(icr_scene *s, const double *f, double *x) {
  auto &F = s->fac;
  const int nc = s->last_build_nc;
  k_gather_fpos<<<cdiv(3 * nc, 256), 256, 0, s->stream>>>(nc, F.d_order, f, F.d_fpos);
  ICR_LAUNCH_CHECK();
  k_zf_part<<<F.n_zf_tasks, 1024, 0, s->stream>>>(F.d_zf_tasks, F.d_sup, F.d_lohi, F.d_Z, F.d_fpos, F.d_zf_part);
  ICR_LAUNCH_CHECK();
  k_zf_sum<<<F.n_zf_sum_tasks, GV_R, 0, s->stream>>>(F.d_zf_tasks, F.d_sup, F.d_lohi, F.d_zf_part, F.d_y);
  ICR_LAUNCH_CHECK();
  backward_solve(s, x);
}

void launch_wh_expand(hipStream_t st, int nc, int nu, const int *idx, const double *w, const double *WN, double *WH) {
  k_wh_expand<<<dim3(cdiv(3L * nc, 256), nc), 256, 0, st>>>(nc, 3 * nu, idx, w, WN, WH);
  ICR_LAUNCH_CHECK();
}

void launch_narrow(icr_scene *s, const double *x, float *y, long n) {
  k_to_float<<<(unsigned)std::min<long>(1024, (n + 255) / 256), 256, 0, s->stream>>>(n, x, y);
  ICR_LAUNCH_CHECK();
}

void launch_widen(icr_scene *s, const float *x, double *y, long n) {
  k_to_double<<<(unsigned)std::min<long>(1024, (n + 255) / 256), 256, 0, s->stream>>>(n, x, y);
  ICR_LAUNCH_CHECK();
}

void launch_fill(icr_scene *s, double *x, long n, double v) {
  k_fill<<<(unsigned)std::min<long>(1024, (n + 255) / 256), 256, 0, s->stream>>>(n, v, x);
  ICR_LAUNCH_CHECK();
}

void ensure_rhs_capacity(icr_scene *s, int nc) {
  auto &F = s->fac;
  if (nc <= F.nc_cap) return;
  s->epoch++;
  ICR_HIP(hipStreamSynchronize(s->stream));
  const bool settled = device_settle();
  F.nc_cap = 0;   // an allocation below may fail
  F.rhs_arena.release(settled);
  long long xo = 0, zo = 0;
  for (int i = 0; i < (int)F.sup.size(); ++i) {
    SupDev &d = F.sup[i];
    int rmax = 3 * std::min(nc, d.region_nodes);
    d.rmax = rmax;
    d.x_off = xo;
    d.z_off = zo;
    xo += (long long)3 * (d.ncol + d.nb) * rmax;
    zo += (long long)3 * d.ncol * rmax;
  }
  F.d_X = F.rhs_arena.alloc<double>(xo);
  F.d_Z = F.rhs_arena.alloc<double>(zo);
  F.x_elems = xo;
  F.z_elems = zo;
  F.mixed_arena.release(settled);   // sized for the previous offsets
  F.mixed_cap = 0;
  {
    // task-list capacities per (level, kind): the counts at r = rmax
    const int nlev = (int)F.levels.size();
    F.rhs_cap.assign(RHS_KINDS * nlev, 0);
    F.rhs_off.assign(RHS_KINDS * nlev, 0);
    std::vector<int> level_first(nlev + 1, 0);
    long long tot = 0;
    for (int l = 0; l < nlev; ++l) {
      const LevelInfo &L = F.levels[l];
      level_first[l] = L.first;
      level_first[l + 1] = L.first + L.count;
      long long mid[RHS_KINDS] = {}, small[RHS_KINDS] = {};
      for (int q = 0; q < L.count; ++q) {
        const SupDev &d = F.sup[F.sym.level_sup[L.first + q]];
        for (int k = 0; k < RHS_KINDS; ++k) {
          mid[k] += rhs_task_count(k, d.rmax, 3 * d.ncol, 3 * d.nb, RHS_T);
          small[k] += rhs_task_count(k, d.rmax, 3 * d.ncol, 3 * d.nb, RHS_TS);
        }
      }
      for (int k = 0; k < RHS_KINDS; ++k) {
        // a list of small tiles has fewer than 4 RHS_SMALL entries
        const long long cap = std::max(mid[k], std::min(small[k], (long long)4 * RHS_SMALL));
        if (cap > INT32_MAX / 2) throw std::runtime_error("multi-RHS task lists exceed 2^30 entries");
        F.rhs_cap[RHS_KINDS * l + k] = (int)cap;
        F.rhs_off[RHS_KINDS * l + k] = (int)tot;
        tot += F.rhs_cap[RHS_KINDS * l + k];
      }
    }
    if (tot > INT32_MAX) throw std::runtime_error("multi-RHS task lists exceed 2^31 entries");
    std::vector<int> asm_first(nlev);
    F.asm_cap = 0;
    for (int l = 0; l < nlev; ++l) {
      asm_first[l] = F.asm_cap;
      F.asm_cap += F.rhs_cap[RHS_KINDS * l + RT_ASM];
    }
    F.d_asm_first = F.rhs_arena.alloc<int>(nlev);
    ICR_HIP(hipMemcpyAsync(F.d_asm_first, asm_first.data(), nlev * sizeof(int), hipMemcpyHostToDevice, s->stream));
    F.d_rhs_tasks = F.rhs_arena.alloc<int2>(std::max<long long>(1, tot));
    F.d_rhs_off = F.rhs_arena.alloc<int>(F.rhs_off.size());
    F.d_rhs_cnt = F.rhs_arena.alloc<int>(F.rhs_off.size());
    F.d_level_first = F.rhs_arena.alloc<int>(level_first.size());
    ICR_HIP(hipMemcpyAsync(F.d_rhs_off, F.rhs_off.data(), F.rhs_off.size() * sizeof(int), hipMemcpyHostToDevice,
                           s->stream));
    ICR_HIP(hipMemcpyAsync(F.d_level_first, level_first.data(), level_first.size() * sizeof(int),
                           hipMemcpyHostToDevice, s->stream));
  }
  const long long m = 3LL * nc;
  F.d_Wp = F.rhs_arena.alloc<double>(m * m);
  F.d_keys = F.rhs_arena.alloc<int>(nc);
  F.d_order = F.rhs_arena.alloc<int>(nc);
  F.d_pos = F.rhs_arena.alloc<int>(nc);
  F.d_lohi = F.rhs_arena.alloc<int>(3LL * F.sup.size());
  F.d_fpos = F.rhs_arena.alloc<double>(3LL * nc);
  F.d_cerr = F.rhs_arena.alloc<int>(1);
  {
    // Z f tasks: one per (supernode, 64-row block, column chunk of ZF_K), the
    // chunk-0 tasks first (they also do the sums); partials per supernode at
    // off_s + chunk * n3 + row
    std::vector<int4> first, rest;
    long long off = 0;
    for (int i = 0; i < (int)F.sup.size(); ++i) {
      const SupDev &d = F.sup[i];
      const int n3 = 3 * d.ncol, nch = std::max(1, cdiv(d.rmax, ZF_K));
      for (int i0 = 0; i0 < n3; i0 += GV_R)
        for (int ch = 0; ch < nch; ++ch) (ch == 0 ? first : rest).push_back(make_int4(i, i0, ch * ZF_K, (int)off));
      off += (long long)n3 * nch;
    }
    F.n_zf_sum_tasks = (int)first.size();
    first.insert(first.end(), rest.begin(), rest.end());
    F.n_zf_tasks = (int)first.size();
    F.d_zf_tasks = F.rhs_arena.alloc<int4>(first.size());
    F.d_zf_part = F.rhs_arena.alloc<double>(std::max<long long>(1, off));
    ICR_HIP(hipMemcpyAsync(F.d_zf_tasks, first.data(), first.size() * sizeof(int4), hipMemcpyHostToDevice,
                           s->stream));
  }
  ICR_HIP(hipMemcpyAsync(F.d_sup, F.sup.data(), F.sup.size() * sizeof(SupDev), hipMemcpyHostToDevice, s->stream));
  ICR_HIP(hipStreamSynchronize(s->stream));
  F.nc_cap = nc;
}

namespace {

// Contact order and the task lists of every tree level (shared by the FP64
// and the mixed-precision builds).
void rhs_prepare(icr_scene *s, int nc, const int *node_ids, bool validate) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  const int nsup = (int)F.sup.size();
  s->last_build_nc = nc;
  if (validate) ICR_HIP(hipMemsetAsync(F.d_cerr, 0, sizeof(int), st));
  k_sort_contacts<<<cdiv(nc, SORT_C), 1024, 0, st>>>(nc, s->mesh.N, nsup, node_ids, F.d_sup_of_node, s->mesh.d_fixed,
                                                     F.d_keys, F.d_order, F.d_pos, F.d_cerr);
  ICR_LAUNCH_CHECK();
  const int nlev = (int)F.levels.size();
  k_rhs_plan<<<dim3(nlev, RHS_KINDS), PLAN_NT, 0, st>>>(nc, F.d_level_first, F.d_level_sup, F.d_sup, F.d_keys, F.d_lohi,
                                                        F.d_rhs_off, F.d_rhs_cnt, F.d_rhs_tasks);
  ICR_LAUNCH_CHECK();
}

// Launch geometry of a product: its list's capacity, one workgroup per task.
struct RhsLists {
  const Factor &F;
  unsigned grid(int l, int k) const { return (unsigned)std::max(1, F.rhs_cap[RHS_KINDS * l + k]); }
  const int2 *list(int l, int k) const { return F.d_rhs_tasks + F.rhs_off[RHS_KINDS * l + k]; }
  const int *count(int l, int k) const { return F.d_rhs_cnt + RHS_KINDS * l + k; }
  bool any(int l, int k) const { return F.rhs_cap[RHS_KINDS * l + k] > 0; }
};

// Z -> Wp, and Wp -> W_H in contact order, FP64 or FP32.
void wh_tiles(icr_scene *s, int nc) {
  auto &F = s->fac;
  auto go = [&](int T, auto kernel) {
    const long nt = cdiv(3L * nc, T), n = nt * (nt + 1) / 2;
    kernel<<<(unsigned)n, 256, 0, s->stream>>>(nc, (int)F.sup.size(), n >= WP_BAND, F.d_sup, F.d_keys, F.d_lohi,
                                                   F.d_anc_ptr, F.d_anc, F.d_Z, F.d_Wp);
  };
  const long nt = cdiv(3L * nc, RHS_T);
  if (nt * (nt + 1) / 2 < WP_SMALL)
    go(RHS_TS, k_wp_tiles<RhsAcc<double>::Small>);
  else
    go(RHS_T, k_wp_tiles<RhsAcc<double>::Mid>);
  ICR_LAUNCH_CHECK();
}
template <class TW>
void wh_finish(icr_scene *s, int nc, TW *WH) {
  k_wh_unpermute<TW><<<3u * nc, 256, 0, s->stream>>>(nc, s->fac.d_pos, s->fac.d_Wp, WH);
  ICR_LAUNCH_CHECK();
}

template <class E>
void rhs_init(icr_scene *s, const int *node_ids, const double *frames, const double *R, E *X) {
  auto &F = s->fac;
  k_rhs_init<E><<<std::max(1, F.asm_cap), 256, 0, s->stream>>>(
      F.d_sup, (int)F.levels.size(), F.d_asm_first, F.d_rhs_off, F.d_rhs_cnt, F.d_rhs_tasks, F.d_child, F.d_invmap_off,
      F.d_invmap, F.d_lohi, F.d_order, node_ids, F.d_iperm, frames, R, X);
  ICR_LAUNCH_CHECK();
}

// One forward sweep over the tree levels in FP32 (the bulk solve of the
// mixed-precision build): X32 from the unit columns (R null) or
// from the residual R and the children, Z32 = L_ss^-1 X32 with its FP64 copy
// stored (z64 = 1) or added (z64 = 2) into Z, X32 below rows -= L_21 Z32.
void forward_fp32(icr_scene *s, const int *node_ids, const double *R, int z64) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  RhsLists L{F};
  rhs_init<float>(s, node_ids, nullptr, R, F.d_X32);
  for (int l = 0; l < (int)F.levels.size(); ++l) {
    if (!L.any(l, RT_ASM)) continue;
    k_rhs_diag<float><<<L.grid(l, RT_DIAG), 256, 0, st>>>(F.d_sup, L.list(l, RT_DIAG), L.count(l, RT_DIAG),
                                                           F.d_lohi, F.d_linv32, F.d_X32, F.d_Z32, F.d_Z, z64);
    ICR_LAUNCH_CHECK();
    if (L.any(l, RT_OFF)) {
      k_rhs_off<float><<<L.grid(l, RT_OFF), 256, 0, st>>>(F.d_sup, L.list(l, RT_OFF), L.count(l, RT_OFF), F.d_lohi,
                                                        F.d_relmap, F.d_front32, F.d_Z32, F.d_X32, R != nullptr);
      ICR_LAUNCH_CHECK();
    }
  }
}

}  // namespace

void ensure_mixed(icr_scene *s) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  if (!F.have32) {
    F.fac32_arena.release(device_settle());
    F.d_front32 = F.fac32_arena.alloc<float>(F.front_elems);
    F.d_linv32 = F.fac32_arena.alloc<float>(F.linv_elems);
    k_to_float<<<2048, 256, 0, st>>>(F.front_elems, F.d_front, F.d_front32);
    ICR_LAUNCH_CHECK();
    k_to_float<<<2048, 256, 0, st>>>(F.linv_elems, F.d_linv, F.d_linv32);
    ICR_LAUNCH_CHECK();
    F.have32 = true;
  }
  if (F.mixed_cap != F.nc_cap) {
    ICR_HIP(hipStreamSynchronize(st));
    F.mixed_cap = 0;   // an allocation below may fail
    F.mixed_arena.release(device_settle());
    F.d_X32 = F.mixed_arena.alloc<float>(F.x_elems);
    F.d_Z32 = F.mixed_arena.alloc<float>(F.z_elems);
    F.d_R = F.mixed_arena.alloc<double>(F.z_elems);
    F.mixed_cap = F.nc_cap;
  }
}

void build_WH_device(icr_scene *s, int nc, const int *node_ids, double *WH, bool validate, const double *frames) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  rhs_prepare(s, nc, node_ids, validate);
  RhsLists L{F};
  rhs_init<double>(s, node_ids, frames, nullptr, F.d_X);
  for (int l = 0; l < (int)F.levels.size(); ++l) {
    if (!L.any(l, RT_ASM)) continue;   // no supernode of the level can hold a contact column
    k_rhs_diag<double><<<L.grid(l, RT_DIAG), 256, 0, st>>>(F.d_sup, L.list(l, RT_DIAG), L.count(l, RT_DIAG), F.d_lohi,
                                                         F.d_linv, F.d_X, F.d_Z, nullptr, 0);
    ICR_LAUNCH_CHECK();
    if (L.any(l, RT_OFF)) {
      k_rhs_off<double><<<L.grid(l, RT_OFF), 256, 0, st>>>(F.d_sup, L.list(l, RT_OFF), L.count(l, RT_OFF), F.d_lohi,
                                                         F.d_relmap, F.d_front, F.d_Z, F.d_X, 0);
      ICR_LAUNCH_CHECK();
    }
  }
  wh_tiles(s, nc);
  wh_finish<double>(s, nc, WH);
}

void build_WH_mixed(icr_scene *s, int nc, const int *node_ids, int refine, float *WH32, double *WH64) {
  auto &F = s->fac;
  hipStream_t st = s->stream;
  rhs_prepare(s, nc, node_ids, false);
  RhsLists L{F};
  forward_fp32(s, node_ids, nullptr, 1);   // Z32 and its FP64 copy Z
  for (int it = 0; it < refine; ++it) {
    // FP64 residual of L Z = P H^T on every supernode's rows, level by level
    rhs_init<double>(s, node_ids, nullptr, nullptr, F.d_X);
    for (int l = 0; l < (int)F.levels.size(); ++l) {
      if (!L.any(l, RT_ASM)) continue;
      k_rhs_resid<<<L.grid(l, RT_DIAG), 256, 0, st>>>(F.d_sup, L.list(l, RT_DIAG), L.count(l, RT_DIAG),
                                                            F.d_lohi, F.d_front, F.d_X, F.d_Z, F.d_R);
      ICR_LAUNCH_CHECK();
      if (L.any(l, RT_OFF)) {
        k_rhs_off<double><<<L.grid(l, RT_OFF), 256, 0, st>>>(F.d_sup, L.list(l, RT_OFF), L.count(l, RT_OFF), F.d_lohi,
                                                           F.d_relmap, F.d_front, F.d_Z, F.d_X, 0);
        ICR_LAUNCH_CHECK();
      }
    }
    forward_fp32(s, node_ids, F.d_R, 2);   // Z += L^-1 R (FP32 solve of the correction)
  }
  wh_tiles(s, nc);   // W_H = Z^T Z in FP64 from the refined Z
  if (WH32) {
    wh_finish<float>(s, nc, WH32);
  }
  if (WH64) {
    wh_finish<double>(s, nc, WH64);
  }
}

}  // namespace icr
