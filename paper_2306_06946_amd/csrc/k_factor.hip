// Supernodal (multifrontal) FP64 Cholesky of A on the device: the factor the
// multi-RHS solves of W_H = H A^-1 H^T run against (Eq. 28).
//
// Fronts are processed by height level of the dissection tree, bottom-up.  A
// level's fronts are assembled together (children's Schur complements pulled
// through index maps, then A's blocks scattered), then partially factored by a
// blocked Cholesky in panels of 256 columns, all fronts of the level in the
// same launches: inside a panel 64 columns at a time, left-looking (the
// panel's earlier columns applied to the tile column, its diagonal tile
// factored and inverted, then the panel solve), after it one update of the
// trailing matrix.  The trailing updates are bound by reading and writing the
// trailing matrix, so one of rank 256 instead of four of rank 64 moves a
// quarter of the bytes.  At the end each supernode's diagonal block inverse
// L_ss^{-1} is formed by doubling (used by the solves as a dense product).
// 61 236 DOF: 6.9 ms; 25.3 ms with panels of 64 columns, a diagonal tile by
// 256 threads with three barriers a column (131 us a tile) and an inverse that
// marched down each tile column (5.9 ms).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "scene.hpp"

namespace icr {

namespace {

// The front's lower triangle from every child's update matrix (its trailing
// Schur complement) through the child's index map; the rest of it is never
// read.  One front per blockIdx.y, one 64 x 64 tile of the lower triangle per
// blockIdx.x; lane = row, wave = 16 columns, whose loads are independent.
// Bound by reading the children and writing the front.
__global__ __launch_bounds__(256) void k_front_init(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                    const int *__restrict__ child, const int *__restrict__ invmap_off,
                                                    const int *__restrict__ invmap, double *__restrict__ front) {
  const SupDev S = sup[level_sup[blockIdx.y]];
  const int f = 3 * (S.ncol + S.nb), nt = (f + TILE - 1) / TILE;
  if ((int)blockIdx.x >= nt * (nt + 1) / 2) return;
  int I, J;
  tri_index(blockIdx.x, I, J);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln = threadIdx.x & 63;
  const int i = TILE * I + ln, j0 = TILE * J + 16 * wv;
  const int ir = min(i, f - 1) / 3, ia = min(i, f - 1) % 3;
  double v[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) v[q] = 0.0;
  for (int c = 0; c < S.nchild; ++c) {
    const int *inv = invmap + invmap_off[S.child_off + c];
    const SupDev C = sup[child[S.child_off + c]];
    const int fc = 3 * (C.ncol + C.nb), n3c = 3 * C.ncol;
    const int ii = inv[ir];
    const double *row = front + C.front_off + (n3c + 3 * ii + ia) + (long)n3c * fc;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int j = j0 + q;
      const int jj = j < f ? inv[j / 3] : -1;
      if (jj >= 0 && ii >= 0 && i >= j) v[q] += row[(long)(3 * jj + j % 3) * fc];
    }
  }
  double *F = front + S.front_off;
#pragma unroll
  for (int q = 0; q < 16; ++q)
    if (i < f && i >= j0 + q) F[i + (long)(j0 + q) * f] = v[q];
}

__global__ void k_front_add_A(const AScatter *__restrict__ list, int count, const SupDev *__restrict__ sup,
                              const double *__restrict__ Ab, double *__restrict__ front) {
  int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= count) return;
  AScatter a = list[e];
  const SupDev S = sup[a.s];
  const int f = 3 * (S.ncol + S.nb);
  double *F = front + S.front_off;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) F[(long)(3 * a.lr + i) + (long)(3 * a.lc + j) * f] += Ab[9L * a.blk + 3 * i + j];
}

// The two wait states between the write of a DPP operand and its use are in the
// statement of the use: the compiler does not know that it has to keep them and
// may put a copy of the operand right before the statement.  One wait covers
// the statement's up to four multiply-adds.
#define ICR_FMAC_BCAST(D, S, B, L) "v_fmac_f64_dpp " D ", " S ", -" B " row_newbcast:" L " row_mask:0xf bank_mask:0xf\n\t"
// a[J + i] -= (lane J + i of this lane's row of 16 of b) * b, 0 <= i < N
template <int J, int N>
__device__ __forceinline__ void fmac_bcast_column(double *a, double b) {
  if constexpr (N == 4)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%4", "%4", "%5") ICR_FMAC_BCAST("%1", "%4", "%4", "%6")
            ICR_FMAC_BCAST("%2", "%4", "%4", "%7") ICR_FMAC_BCAST("%3", "%4", "%4", "%8")
        : "+&v"(a[J]), "+&v"(a[J + 1]), "+&v"(a[J + 2]), "+&v"(a[J + 3])
        : "v"(b), "n"(J), "n"(J + 1), "n"(J + 2), "n"(J + 3));
  else if constexpr (N == 3)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%3", "%3", "%4") ICR_FMAC_BCAST("%1", "%3", "%3", "%5")
            ICR_FMAC_BCAST("%2", "%3", "%3", "%6")
        : "+&v"(a[J]), "+&v"(a[J + 1]), "+&v"(a[J + 2])
        : "v"(b), "n"(J), "n"(J + 1), "n"(J + 2));
  else if constexpr (N == 2)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%2", "%2", "%3") ICR_FMAC_BCAST("%1", "%2", "%2", "%4")
        : "+&v"(a[J]), "+&v"(a[J + 1])
        : "v"(b), "n"(J), "n"(J + 1));
  else if constexpr (N == 1)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%1", "%1", "%2") : "+&v"(a[J]) : "v"(b), "n"(J));
}
// s -= sum over 0 <= i < N, in order, of (lane LANE of this lane's row of 16 of a[i]) * x[i]
template <int LANE, int N>
__device__ __forceinline__ void fmac_bcast_row(double &s, const double *a, const double *x) {
  if constexpr (N == 4)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%1", "%5", "%9") ICR_FMAC_BCAST("%0", "%2", "%6", "%9")
            ICR_FMAC_BCAST("%0", "%3", "%7", "%9") ICR_FMAC_BCAST("%0", "%4", "%8", "%9")
        : "+&v"(s)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "n"(LANE));
  else if constexpr (N == 3)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%1", "%4", "%7") ICR_FMAC_BCAST("%0", "%2", "%5", "%7")
            ICR_FMAC_BCAST("%0", "%3", "%6", "%7")
        : "+&v"(s)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "n"(LANE));
  else if constexpr (N == 2)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%1", "%3", "%5") ICR_FMAC_BCAST("%0", "%2", "%4", "%5")
        : "+&v"(s)
        : "v"(a[0]), "v"(a[1]), "v"(x[0]), "v"(x[1]), "n"(LANE));
  else if constexpr (N == 1)
    asm("s_nop 1\n\t" ICR_FMAC_BCAST("%0", "%1", "%2", "%3") : "+&v"(s) : "v"(a[0]), "v"(x[0]), "n"(LANE));
}
#undef ICR_FMAC_BCAST
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int LANE>
__device__ __forceinline__ double lane_value(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, LANE), hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), LANE);
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// 1 / sqrt(x) from the hardware estimate refined by two Newton steps.
__device__ __forceinline__ double rsqrt2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}

constexpr int PD = 65;   // LDS row stride of a 64 x 64 tile

// Cholesky factor of the 16 x 16 block D (row stride PD, lower) in place and
// its inverse to X, by one wave: lane l holds row l % 16 in registers (the
// four rows of 16 lanes repeat the same work).  A column's multipliers reach
// the other rows through the broadcast of the multiply-add itself, so a column
// costs one instruction per remaining column.  bad: first column without a
// positive pivot, or 16.
__device__ __forceinline__ int potrf16(double *D, double *X) {
  const int l = threadIdx.x & 15;
  double a[16], r[16];
  int bad = 16;
#pragma unroll
  for (int c = 0; c < 16; ++c) a[c] = D[l * PD + c];
  static_for<0, 16>([&](auto cc) {
    constexpr int c = decltype(cc)::value;
    double d = lane_value<c>(a[c]);
    if (!(d > 0.0)) {
      bad = min(bad, c);
      d = 1.0;
    }
    r[c] = rsqrt2(d);
    const double lc = l > c ? a[c] * r[c] : l == c ? d * r[c] : 0.0;
    a[c] = lc;
    static_for<0, (15 - c + 3) / 4>([&](auto gg) {
      constexpr int j = c + 1 + 4 * decltype(gg)::value;
      fmac_bcast_column<j, j + 4 <= 16 ? 4 : 16 - j>(a, lc);
    });
  });
  // column l of the inverse: x_i = (delta_il - sum_{q<i} L(i, q) x_q) / L(i, i)
  double x[16];
  static_for<0, 16>([&](auto ii) {
    constexpr int i = decltype(ii)::value;
    double s = l == i ? 1.0 : 0.0;
    static_for<0, (i + 3) / 4>([&](auto gg) {
      constexpr int q = 4 * decltype(gg)::value;
      fmac_bcast_row<i, q + 4 <= i ? 4 : i - q>(s, a + q, x + q);
    });
    x[i] = s * r[i];
  });
  if ((threadIdx.x & 63) < 16) {
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      D[l * PD + c] = a[c];
      X[c * PD + l] = x[c];
    }
  }
  return bad;
}

// c +- A B of 16 x 16 LDS blocks (one wave); TB: B transposed.
template <bool TB>
__device__ __forceinline__ mfma_d4 mma16(const double *A, const double *B, mfma_d4 c) {
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
#pragma unroll
  for (int k = 0; k < 16; k += 4)
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(A[li * PD + k + lk], TB ? B[li * PD + k + lk] : B[(k + lk) * PD + li], c,
                                             0, 0, 0);
  return c;
}
// D(i, j) of the accumulator: lane j + 16 (i % 4), register i / 4
template <class F>
__device__ __forceinline__ void acc16(F &&f) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < 4; ++t) f(4 * t + (l >> 4), l & 15, t);
}

// Tile column k of the panel that starts at column kp, every front of the
// level: the panel's columns kp .. k - 1 applied to its row tiles, and (row
// tile 0) the diagonal tile factored and its inverse written into the diagonal
// tile of L_ss^{-1} (upper part zero).  The diagonal tile goes by 16 x 16
// blocks in LDS: one wave factors and inverts a diagonal block, the products
// are MFMAs spread over the four waves.  28 us a launch, most of it the latency
// of 64 dependent pivots.
__global__ __launch_bounds__(256) void k_panel_tile(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                    int kp, int k, double *__restrict__ front,
                                                    double *__restrict__ linv, int *__restrict__ err) {
  __shared__ double D[64 * PD];
  __shared__ double X[64 * PD];   // the inverse; before, the staging of the update
  static_assert(AccS::LDS <= 64 * PD, "staging fits the inverse's tile");
  const SupDev S = sup[level_sup[blockIdx.y]];
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  if (k >= n3) return;
  const int t = min(64, n3 - k);
  const int i0 = k + TILE * blockIdx.x;
  if (i0 >= f || (blockIdx.x > 0 && k == kp)) return;
  double *F = front + S.front_off;
  const int M = min(TILE, f - i0);
  const int tid = threadIdx.x, wv = tid >> 6;
  AccS acc;
  acc.zero();
  if (k > kp)
    acc.acc<true, true>(F + k + (long)kp * f, f, F + i0 + (long)kp * f, f, t, M, 0, k - kp, X);
  // the accumulator holds the tile transposed: its lanes then run along the
  // rows of the column-major front
  if (blockIdx.x > 0) {
    double *P = F + i0 + (long)k * f;
    acc.update(P, f, P, f, t, M, [](int, int) { return true; }, [](int, int, double v, double old) { return old - v; });
    return;
  }
  // the diagonal tile, padded to 64 by the identity (a row tile holds rows
  // beyond it when t < 64)
  acc.for_each([&](int j, int i, double v) {
    D[i * PD + j] = (i < t && j < t) ? (i >= j ? F[(long)(k + i) + (long)(k + j) * f] - v : 0.0) : (i == j ? 1.0 : 0.0);
    if (i >= t && i < M && j < t) F[(long)(k + i) + (long)(k + j) * f] -= v;
  });
  __syncthreads();
  for (int b = 0; b < 4; ++b) {
    double *Db = D + 16 * b * (PD + 1);
    if (wv == 0) {
      const int bad = potrf16(Db, X + 16 * b * (PD + 1));
      if (tid == 0 && bad < 16) atomicMin(err, 3 * S.col0 + k + 16 * b + bad);
    }
    __syncthreads();
    if (wv > b) {   // block row wv below: P = A X_b^T
      double *P = D + 16 * wv * PD + 16 * b;
      const mfma_d4 c = mma16<true>(P, X + 16 * b * (PD + 1), mfma_d4{0.0, 0.0, 0.0, 0.0});
      acc16([&](int i, int j, int r) { P[i * PD + j] = c[r]; });
    }
    __syncthreads();
    for (int q = wv; q < (3 - b) * (4 - b) / 2; q += 4) {   // A(I, J) -= P_I P_J^T
      int I = b + 1, J = q;
      while (J > I - b - 1) {
        J -= I - b;
        ++I;
      }
      J += b + 1;
      const mfma_d4 c = mma16<true>(D + 16 * I * PD + 16 * b, D + 16 * J * PD + 16 * b, mfma_d4{0.0, 0.0, 0.0, 0.0});
      acc16([&](int i, int j, int r) { D[(16 * I + i) * PD + 16 * J + j] -= c[r]; });
    }
    __syncthreads();
  }
  // block column wv of the inverse: X(I, J) = -X(I, I) sum_{J<=K<I} L(I, K) X(K, J)
  for (int I = 0; I < 4; ++I) {
    double *XI = X + 16 * I * PD + 16 * wv;
    if (I < wv) {
      acc16([&](int i, int j, int) { XI[i * PD + j] = 0.0; });
    } else if (I > wv) {
      mfma_d4 c = {0.0, 0.0, 0.0, 0.0};
      for (int K = wv; K < I; ++K) c = mma16<false>(D + 16 * I * PD + 16 * K, X + 16 * K * PD + 16 * wv, c);
      acc16([&](int i, int j, int r) { XI[i * PD + j] = c[r]; });
      __builtin_amdgcn_wave_barrier();
      __threadfence_block();
      c = mma16<false>(X + 16 * I * (PD + 1), XI, mfma_d4{0.0, 0.0, 0.0, 0.0});
      __builtin_amdgcn_wave_barrier();
      __threadfence_block();
      acc16([&](int i, int j, int r) { XI[i * PD + j] = -c[r]; });
    }
    __syncthreads();
  }
  double *Li = linv + S.linv_off;
  for (int e = tid; e < 64 * 64; e += 256) {
    const int i = e & 63, j = e >> 6;
    if (i >= t || j >= t) continue;
    if (i >= j) F[(long)(k + i) + (long)(k + j) * f] = D[i * PD + j];
    Li[(long)(k + i) + (long)(k + j) * n3] = i >= j ? X[i * PD + j] : 0.0;
  }
}

// Panel rows below the diagonal tile: P <- P D^{-T} (the accumulator holds the
// tile transposed, as above).
__global__ __launch_bounds__(256) void k_trsm_panel(const SupDev *__restrict__ sup,
                                                    const int *__restrict__ level_sup, int k,
                                                    double *__restrict__ front, const double *__restrict__ linv) {
  __shared__ double lds[AccS::LDS];
  const SupDev S = sup[level_sup[blockIdx.y]];
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  if (k >= n3) return;
  const int t = min(64, n3 - k);
  const int i0 = k + t + TILE * blockIdx.x;
  if (i0 >= f) return;
  const int M = min(TILE, f - i0);
  double *F = front + S.front_off;
  const double *Di = linv + S.linv_off + k + (long)k * n3;
  AccS acc;
  acc.zero();
  // out(j, i) = sum_c Dinv(j, c) P(i, c)
  acc.acc<true, true>(Di, n3, F + i0 + (long)k * f, f, t, M, 0, t, lds);
  acc.put(F + i0 + (long)k * f, f, t, M, [](double v) { return v; });
}

// Trailing update of the lower triangle by the panel of up to FP_W columns at
// kp: F(i, j) -= sum_c P(i, c) P(j, c).
constexpr int FP_W = 256;
__global__ __launch_bounds__(256) void k_trailing(const SupDev *__restrict__ sup, const int *__restrict__ level_sup,
                                                  int kp, double *__restrict__ front) {
  __shared__ double lds[AccS::LDS];
  const SupDev S = sup[level_sup[blockIdx.y]];
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  if (kp >= n3) return;
  const int w = min(FP_W, n3 - kp);
  const int base = kp + w;
  const int rem = f - base;
  if (rem <= 0) return;
  const int nt = (rem + TILE - 1) / TILE;
  if ((int)blockIdx.x >= nt * (nt + 1) / 2) return;
  int I, J;
  tri_index(blockIdx.x, I, J);
  const int i0 = base + TILE * I, j0 = base + TILE * J;
  const int M = min(TILE, f - i0), N = min(TILE, f - j0);
  double *F = front + S.front_off;
  AccS acc;
  acc.zero();
  acc.acc<true, true>(F + j0 + (long)kp * f, f, F + i0 + (long)kp * f, f, N, M, 0, w, lds);
  double *C = F + i0 + (long)j0 * f;
  acc.update(C, f, C, f, N, M, [&](int j, int i) { return i0 + i >= j0 + j; },
             [](int, int, double v, double old) { return old - v; });
}

// L_ss^{-1} by doubling, from the inverses of the diagonal tiles: with the
// diagonal blocks A and C of h tiles inverted, the block below A is
// -C^{-1} (L_21 A^{-1}).  One workgroup per tile (I, J) of that block, all
// supernodes with more than h tiles (sup_by_tiles: by descending tile count)
// in one launch per product, so the number of launches is twice the logarithm
// of the largest tile count.  The product L_21 A^{-1} is kept, transposed, in
// the mirror tile (J, I) of L_ss^{-1}, whose strictly upper tiles are never
// read by the solves.
__global__ __launch_bounds__(256) void k_linv(const SupDev *__restrict__ sup, const int *__restrict__ sup_by_tiles,
                                              int nsup, int h, int second, const double *__restrict__ front,
                                              double *__restrict__ linv) {
  __shared__ double lds[AccS::LDS];
  const SupDev S = sup[sup_by_tiles[blockIdx.x % nsup]];
  const int tile = blockIdx.x / nsup;
  const int n3 = 3 * S.ncol, f = 3 * (S.ncol + S.nb);
  const int T = (n3 + TILE - 1) / TILE;
  const int r0 = 2 * h * (tile / (h * h)), q = tile % (h * h);
  const int I = r0 + h + q / h, J = r0 + q % h;
  if (I >= T) return;
  double *X = linv + S.linv_off;
  const int i0 = TILE * I, j0 = TILE * J, m0 = TILE * (r0 + h);
  const int M = min(TILE, n3 - i0);
  AccS acc;
  acc.zero();
  if (!second) {
    acc.acc<true, false>(front + S.front_off + i0, f, X + (long)j0 * n3, n3, M, TILE, j0, m0, lds);
    acc.put(X + j0 + (long)i0 * n3, n3, M, TILE, [](double v) { return v; });
  } else {
    acc.acc<true, true>(X + j0, n3, X + i0, n3, TILE, M, m0, i0 + M, lds);
    acc.put(X + i0 + (long)j0 * n3, n3, TILE, M, [](double v) { return -v; });
  }
}

}  // namespace

void run_numeric_factor(icr_scene *s) {
  auto &F = s->fac;
  auto &m = s->mesh;
  hipStream_t st = s->stream;
  ICR_HIP(hipMemsetAsync(F.d_err, 0x7f, sizeof(int), st));
  hipEvent_t e0, e1;
  ICR_HIP(hipEventCreate(&e0));
  ICR_HIP(hipEventCreate(&e1));
  ICR_HIP(hipEventRecord(e0, st));
  for (size_t l = 0; l < F.levels.size(); ++l) {
    const LevelInfo &L = F.levels[l];
    if (L.count == 0) continue;
    const int *lsup = F.d_level_sup + L.first;
    const int ft = cdiv(L.max_f3, TILE);
    k_front_init<<<dim3(ft * (ft + 1) / 2, L.count), 256, 0, st>>>(F.d_sup, lsup, F.d_child, F.d_invmap_off,
                                                                   F.d_invmap, F.d_front);
    ICR_LAUNCH_CHECK();
    if (L.a_count > 0) {
      k_front_add_A<<<cdiv(L.a_count, 256), 256, 0, st>>>(F.d_ascat + L.a_first, L.a_count, F.d_sup, m.d_A,
                                                          F.d_front);
      ICR_LAUNCH_CHECK();
    }
    for (int kp = 0; kp < L.max_n3; kp += FP_W) {
      for (int k = kp; k < std::min(kp + FP_W, L.max_n3); k += TILE) {
        const int rows = cdiv(L.max_f3 - k, TILE);   // row tiles from the diagonal one down, at most
        k_panel_tile<<<dim3(k == kp ? 1 : rows, L.count), 256, 0, st>>>(F.d_sup, lsup, kp, k, F.d_front, F.d_linv,
                                                                        F.d_err);
        ICR_LAUNCH_CHECK();
        k_trsm_panel<<<dim3(rows, L.count), 256, 0, st>>>(F.d_sup, lsup, k, F.d_front, F.d_linv);
        ICR_LAUNCH_CHECK();
      }
      if (L.max_f3 > kp) {
        const int pt = cdiv(L.max_f3 - kp, TILE);   // upper bound of the trailing row tiles
        k_trailing<<<dim3(pt * (pt + 1) / 2, L.count), 256, 0, st>>>(F.d_sup, lsup, kp, F.d_front);
        ICR_LAUNCH_CHECK();
      }
    }
  }
  for (int h = 1; h < F.max_tiles; h *= 2) {
    int n = 0;   // supernodes with more than h tiles
    while (n < (int)F.tiles_desc.size() && F.tiles_desc[n] > h) ++n;
    const unsigned gx = (unsigned)(cdiv(F.max_tiles, 2 * h) * h * h);
    for (int second = 0; second < 2; ++second) {
      k_linv<<<gx * n, 256, 0, st>>>(F.d_sup, F.d_sup_by_tiles, n, h, second, F.d_front, F.d_linv);
      ICR_LAUNCH_CHECK();
    }
  }
  ICR_HIP(hipEventRecord(e1, st));
  ICR_HIP(hipEventSynchronize(e1));
  float ms = 0;
  ICR_HIP(hipEventElapsedTime(&ms, e0, e1));
  F.ms = ms;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
}

}  // namespace icr
