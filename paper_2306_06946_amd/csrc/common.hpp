// Device-side helpers shared by the library's kernels: error checking, the
// FP64 LDS-tiled GEMM tile used by the supernodal factor and solves.
#pragma once

#include <hip/hip_runtime.h>

#include <stdexcept>
#include <string>

#include "icr_internal.hpp"

namespace icr {

struct HipError : std::runtime_error {
  hipError_t code;
  HipError(hipError_t c, const std::string &where)
      : std::runtime_error(where + ": " + hipGetErrorString(c)), code(c) {}
};

#define ICR_HIP(call)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess) throw ::icr::HipError(e_, std::string(#call) + " @" + __FILE__ + \
                                                   ":" + std::to_string(__LINE__));     \
  } while (0)

#define ICR_LAUNCH_CHECK() ICR_HIP(hipGetLastError())

constexpr int TILE = 64;   // output tile edge of the FP64 GEMM tiles
constexpr int KT = 16;     // K-chunk staged in LDS per iteration

typedef double mfma_d4 __attribute__((ext_vector_type(4)));
typedef float mfma_f4 __attribute__((ext_vector_type(4)));

// One 16x16x4 MFMA per element type: FP64 (v_mfma_f64_16x16x4f64) or FP32
// (v_mfma_f32_16x16x4f32).  Both take A(i, k) from lane i + 16 k and B(k, j)
// from lane j + 16 k; they differ in where D(i, j) lands (checked on gfx950):
// FP64 in lane j + 16 (i % 4), register i / 4; FP32 in lane j + 16 (i / 4),
// register i % 4.
template <class T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef mfma_d4 V;
  __device__ static V op(double a, double b, V c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return 4 * r + (lane >> 4); }
};
template <>
struct Mfma<float> {
  typedef mfma_f4 V;
  __device__ static V op(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Raw buffer access: an 8- or 4-byte element at a byte offset from a uniform
// base; a load at or past num_bytes returns zero, a store there is dropped, so
// an edge needs no branch.  BUF_OUT is past the end of every buffer made here
// (num_bytes < 2^31), also with a further offset below 2^31 added.
typedef unsigned buf_u32x2 __attribute__((ext_vector_type(2)));
constexpr unsigned BUF_OUT = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_make(const void *p, long num_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)num_bytes, 0x00027000);
}
template <class E>
__device__ __forceinline__ E buf_load(__amdgpu_buffer_rsrc_t r, unsigned off);
template <>
__device__ __forceinline__ double buf_load<double>(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(double, (buf_u32x2)__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <>
__device__ __forceinline__ float buf_load<float>(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(float, (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, double v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(buf_u32x2, v), r, off, 0, 0);
}
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, unsigned off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, 0);
}

// Generalised MFMA tile: 4 waves as 2x2, each (16 WB) x (16 WB) of 16x16
// blocks, output tile T = 32 WB, element type E (double or float, operands
// and accumulation alike).  The K-chunk of A (T x KC) and B (KC x T) is
// staged in LDS as [k][i] / [k][j] rows padded to T + 1 elements (no bank
// conflicts for either staging order or the MFMA operand reads), the next
// chunk is prefetched into registers while the MFMAs of the current one run.
// An FP64 MFMA holds its SIMD's vector unit for 64 cycles, so every other
// vector instruction of the loop costs matrix rate: the staging addresses are
// byte offsets kept in registers, the chunks advance the uniform base, and
// the edges are the buffers' ends.  Z^T Z of 9000 columns and 2520 rows:
// 3.92 ms with a bounds check and an address per load, 3.61 ms now (the matrix
// unit busy 88 % of the time).
template <int WB, int KC = KT, class E = double>
struct AccMT {
  typedef E elem;
  typedef typename Mfma<E>::V V;
  static constexpr int T = 32 * WB;
  static constexpr int TP = T + 1;
  static constexpr int NE = T * KC / 256;   // staged elements per thread and operand
  static constexpr int LDS = 2 * KC * TP;   // elements of LDS
  V c[WB][WB];
  __device__ void zero() {
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b) c[a][b] = V{0, 0, 0, 0};
  }
  // One operand's staging.  Thread tid stages, for every q < NE, element
  // (i, k): with rows contiguous (F) i = tid % T, k = tid / T + q (256 / T);
  // else k = tid % KC, i = tid / KC + q (256 / KC).
  template <bool F>
  struct Stage {
    const E *p;         // element (0, kb) of the chunk at hand
    long ld;
    int n;              // valid i
    int i, k;           // of q = 0
    unsigned off[NE];   // byte offset of element q from p, BUF_OUT at an i that the buffer's end does not catch
    // i0: the operand's first row is the tile's row i0 (rows before it are
    // zero: their offsets wrap past every buffer's end; rows not contiguous)
    __device__ __forceinline__ Stage(const E *P, long ld_, int n_, int k0, int i0 = 0) : ld(ld_), n(n_) {
      const int tid = threadIdx.x;
      i = F ? tid % T : tid / KC;
      k = F ? tid / T : tid % KC;
      p = P + (F ? k0 * ld : (long)k0);
#pragma unroll
      for (int q = 0; q < NE; ++q)
        off[q] = (unsigned)sizeof(E) * (F ? (unsigned)i + (unsigned)(k + 256 / T * q) * (unsigned)ld
                                          : (unsigned)k + (unsigned)(i - i0 + 256 / KC * q) * (unsigned)ld);
      if (F && i >= n)
#pragma unroll
        for (int q = 0; q < NE; ++q) off[q] = BUF_OUT;
    }
    // the chunk of kc <= KC columns at p (zeros if kc <= 0)
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk(int kc) const {
      return buf_make(p, kc <= 0 ? 0L : (long)sizeof(E) * (F ? (long)(kc - 1) * ld + n : (long)(n - 1) * ld + kc));
    }
    __device__ __forceinline__ E load(__amdgpu_buffer_rsrc_t b, int kc, int q) const {
      return buf_load<E>(b, !F && k >= kc ? BUF_OUT : off[q]);   // rows contiguous: past the buffer's end
    }
    __device__ __forceinline__ void load(E (&r)[NE], int kc) const {
      const __amdgpu_buffer_rsrc_t b = chunk(kc);
#pragma unroll
      for (int q = 0; q < NE; ++q) r[q] = load(b, kc, q);
    }
    __device__ __forceinline__ void next() { p += F ? KC * ld : (long)KC; }
    __device__ __forceinline__ void store(const E (&r)[NE], E *lds) const {
#pragma unroll
      for (int q = 0; q < NE; ++q) lds[(F ? (k + 256 / T * q) * TP + i : k * TP + i + 256 / KC * q)] = r[q];
    }
  };
  // c += A(i, k) B(k, j) over k in [k0, k1), rows i < M and columns j < N of
  // the tile (M, N >= 1); A(i, k) = A[i + k lda] with AF, A[i lda + k] without
  // (lda >= k1 then), B(k, j) = B[j + k ldb] with BF, B[j ldb + k] without.
  // TRI: B is the transpose of a lower triangle, B(k, j) = 0 for k > j + tri.
  template <bool AF, bool BF, bool TRI = false>
  __device__ void acc(const E *A, long lda, const E *B, long ldb, int M, int N, int k0, int k1, E *lds, int tri = 0) {
    static_assert(!TRI || BF, "a triangle is staged with its columns contiguous");
    if (k0 >= k1) return;
    Stage<AF> sa(A, lda, M, k0);
    Stage<BF> sb(B, ldb, N, k0);
    E ra[NE], rb[NE];
    sa.load(ra, min(KC, k1 - k0));
    sb.load(rb, min(KC, k1 - k0));
    for (int kb = k0; kb < k1; kb += KC) {
      if (TRI && kb + KC - 1 > tri)
#pragma unroll
        for (int q = 0; q < NE; ++q)
          if (kb + sb.k + 256 / T * q > sb.i + tri) rb[q] = E(0);
      sa.store(ra, lds);
      sb.store(rb, lds + KC * TP);
      __syncthreads();
      sa.next();
      sb.next();
      products(lds, KC, sa, ra, sb, rb, min(KC, k1 - kb - KC));
      __syncthreads();
    }
  }
  // c += the staged chunk, its first have columns (in sixteens), and the loads
  // of the next chunk of kc columns.  In the 64 x 64 FP64 tile they are spread
  // over the products: a wave issues in order, and 16 loads in a row keep it
  // from its first product (W_H of 1000 contacts 2.01 -> 1.96 ms, of 3000 9.67
  // -> 9.53; the 32 x 32 tile, one product a step, and FP32 were 1 to 4 %
  // slower with it).
  template <class SA, class SB>
  __device__ __forceinline__ void products(const E *lds, int have, const SA &sa, E (&ra)[NE], const SB &sb, E (&rb)[NE],
                                           int kc) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r0 = (T / 2) * (w >> 1), c0 = (T / 2) * (w & 1);
    const int li = l & 15, lk = l >> 4;
    if constexpr (WB == 1 || sizeof(E) == 4) {
      if (kc > 0) {
        sa.load(ra, kc);
        sb.load(rb, kc);
      }
#pragma unroll
      for (int kk = 0; kk < KC; kk += 4) {
        if (kk % 16 == 0 && kk >= have) break;
        const int k = kk + lk;
        E av[WB], bv[WB];
#pragma unroll
        for (int a = 0; a < WB; ++a) av[a] = lds[k * TP + r0 + 16 * a + li];
#pragma unroll
        for (int b = 0; b < WB; ++b) bv[b] = lds[KC * TP + k * TP + c0 + 16 * b + li];
#pragma unroll
        for (int a = 0; a < WB; ++a)
#pragma unroll
          for (int b = 0; b < WB; ++b) c[a][b] = Mfma<E>::op(av[a], bv[b], c[a][b]);
      }
      return;
    }
    constexpr int STEPS = KC / 4, PER = 2 * NE / STEPS;   // loads per step
    static_assert(PER * STEPS == 2 * NE && KC % 16 == 0, "loads spread evenly");
    const __amdgpu_buffer_rsrc_t ba = sa.chunk(kc), bb = sb.chunk(kc);
    auto loads = [&](int s) {
#pragma unroll
      for (int q = s * PER; q < (s + 1) * PER; ++q) {
        if (q < NE)
          ra[q] = sa.load(ba, kc, q);
        else
          rb[q - NE] = sb.load(bb, kc, q - NE);
      }
    };
    E av[2][WB], bv[2][WB];
    auto read = [&](int s, int z) {
      const int k = 4 * s + lk;
#pragma unroll
      for (int a = 0; a < WB; ++a) av[z][a] = lds[k * TP + r0 + 16 * a + li];
#pragma unroll
      for (int b = 0; b < WB; ++b) bv[z][b] = lds[KC * TP + k * TP + c0 + 16 * b + li];
    };
#pragma unroll
    for (int g = 0; g < STEPS; g += 4) {
      if (4 * g < have) {
        read(g, 0);
#pragma unroll
        for (int s = g; s < g + 4; ++s) {
          if (s + 1 < g + 4) read(s + 1, (s + 1) & 1);
          loads(s);
#pragma unroll
          for (int a = 0; a < WB; ++a)
#pragma unroll
            for (int b = 0; b < WB; ++b) c[a][b] = Mfma<E>::op(av[s & 1][a], bv[s & 1][b], c[a][b]);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int s = g; s < g + 4; ++s) loads(s);
      }
    }
  }
  // c += sum over q < n of A_q^T B_q; get(q, A, an, as, B, bn, bs, rows) names
  // the an columns at A, of that many rows, that meet the tile from its row as
  // on, and the bn at B from its column bs.  The staging runs ahead across q.
  template <class G>
  __device__ void chain_product(int n, G &&get, E *lds) {
    const E *A, *B;
    int an, as, bn, bs, left, q = 0;
    get(0, A, an, as, B, bn, bs, left);
    Stage<false> sa(A, left, an, 0, as), sb(B, left, bn, 0, bs);
    E ra[NE], rb[NE];
    int kc = min(KC, left);
    sa.load(ra, kc);
    sb.load(rb, kc);
    while (q < n) {
      const int have = kc;
      sa.store(ra, lds);
      sb.store(rb, lds + KC * TP);
      __syncthreads();
      left -= kc;
      if (left > 0) {
        sa.next();
        sb.next();
      } else if (++q < n) {
        get(q, A, an, as, B, bn, bs, left);
        sa = Stage<false>(A, left, an, 0, as);
        sb = Stage<false>(B, left, bn, 0, bs);
      }
      kc = q < n ? min(KC, left) : 0;
      products(lds, have, sa, ra, sb, rb, kc);
      __syncthreads();
    }
  }
  template <class F>
  __device__ void for_each(F &&f) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r0 = (T / 2) * (w >> 1), c0 = (T / 2) * (w & 1);
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) f(r0 + 16 * a + Mfma<E>::row(l, t), c0 + 16 * b + (l & 15), c[a][b][t]);
  }
  // C[i ld + j] = f(i, j, v, Q[i ldq + j]) for the tile's i < M, j < N where
  // keep(i, j); every element of Q is loaded before the first is used, and no
  // branch is taken (ld, ldq >= N).
  template <class P, class O, class K, class F>
  __device__ void update(O *C, long ld, const P *Q, long ldq, int M, int N, K &&keep, F &&f) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r0 = (T / 2) * (w >> 1), c0 = (T / 2) * (w & 1) + (l & 15);
    const __amdgpu_buffer_rsrc_t bc = buf_make(C, (long)sizeof(O) * ((M - 1) * ld + N));
    const __amdgpu_buffer_rsrc_t bq = buf_make(Q, (long)sizeof(P) * ((M - 1) * ldq + N));
    P old[WB][WB][4];
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = r0 + 16 * a + Mfma<E>::row(l, t), j = c0 + 16 * b;
          old[a][b][t] = buf_load<P>(
              bq, j < N && keep(i, j) ? (unsigned)sizeof(P) * ((unsigned)i * (unsigned)ldq + (unsigned)j) : BUF_OUT);
        }
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = r0 + 16 * a + Mfma<E>::row(l, t), j = c0 + 16 * b;
          buf_store(bc, j < N && keep(i, j) ? (unsigned)sizeof(O) * ((unsigned)i * (unsigned)ld + (unsigned)j) : BUF_OUT,
                    (O)f(i, j, c[a][b][t], old[a][b][t]));
        }
  }
  // C[i ld + row(j)] = Q[i ldq + j] - v, or the sum of that and what is there
  // (add), for the tile's i < M, j < N (row(j) < ld, ldq >= N)
  template <class R>
  __device__ void push(E *C, long ld, R &&row, const E *Q, long ldq, int M, int N, bool add) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r0 = (T / 2) * (w >> 1), c0 = (T / 2) * (w & 1) + (l & 15);
    const __amdgpu_buffer_rsrc_t bc = buf_make(C, (long)sizeof(E) * M * ld);
    const __amdgpu_buffer_rsrc_t bq = buf_make(Q, (long)sizeof(E) * ((M - 1) * ldq + N));
    unsigned at[WB];
    E q[WB][WB][4];
#pragma unroll
    for (int b = 0; b < WB; ++b) at[b] = c0 + 16 * b < N ? (unsigned)sizeof(E) * (unsigned)row(c0 + 16 * b) : BUF_OUT;
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = r0 + 16 * a + Mfma<E>::row(l, t), j = c0 + 16 * b;
          q[a][b][t] =
              buf_load<E>(bq, j < N ? (unsigned)sizeof(E) * ((unsigned)i * (unsigned)ldq + (unsigned)j) : BUF_OUT) -
              c[a][b][t];
        }
    if (add)
#pragma unroll
      for (int a = 0; a < WB; ++a)
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
          for (int t = 0; t < 4; ++t)
            q[a][b][t] += buf_load<E>(
                bc, (unsigned)sizeof(E) * (unsigned)(r0 + 16 * a + Mfma<E>::row(l, t)) * (unsigned)ld + at[b]);
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          buf_store(bc, (unsigned)sizeof(E) * (unsigned)(r0 + 16 * a + Mfma<E>::row(l, t)) * (unsigned)ld + at[b],
                    q[a][b][t]);
  }
  // C[i ld + j] = f(v) for the tile's i < M, j < N
  template <class O, class F>
  __device__ void put(O *C, long ld, int M, int N, F &&f) {
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int r0 = (T / 2) * (w >> 1), c0 = (T / 2) * (w & 1) + (l & 15);
    const __amdgpu_buffer_rsrc_t bc = buf_make(C, (long)sizeof(O) * ((M - 1) * ld + N));
#pragma unroll
    for (int a = 0; a < WB; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = r0 + 16 * a + Mfma<E>::row(l, t), j = c0 + 16 * b;
          buf_store(bc, j < N ? (unsigned)sizeof(O) * ((unsigned)i * (unsigned)ld + (unsigned)j) : BUF_OUT,
                    (O)f(c[a][b][t]));
        }
  }
};
typedef AccMT<2, 32> AccS;          // 64 x 64 FP64, K-chunk 32

// Lower-triangle tile index x -> (I, J), I >= J, row-major over the triangle.
__device__ inline void tri_index(int x, int &I, int &J) {
  int i = (int)((sqrt(8.0 * (double)x + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= x) ++i;
  while (i * (i + 1) / 2 > x) --i;
  I = i;
  J = x - i * (i + 1) / 2;
}

inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }

}  // namespace icr
