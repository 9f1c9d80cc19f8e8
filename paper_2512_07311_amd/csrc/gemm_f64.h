// Complex fp64 tile GEMM engine on CDNA matrix cores (v_mfma_f64_16x16x4f64).
//
// One workgroup computes a 64x64 complex output tile; its waves form a
// 2 x GT_WN grid, each owning a 32 x (64 / GT_WN) part as 16x16 MFMA blocks
// with separate real and imaginary accumulators.  A complex product is four
// real MFMAs:  Cr += Ar Br - Ai Bi,  Ci += Ar Bi + Ai Br, in ascending k, so
// an output element's rounding does not depend on the tiling.
//
// MFMA f64 16x16x4 operand layout (lane l of 64):
//   A (16x4):  A[l % 16][l / 16]      B (4x16): B[l / 16][l % 16]
//   D (16x16): D[(l / 16) + 4 r][l % 16], r = 0..3 in the four result regs
//   (measured on gfx950; the fp32/bf16 16x16 forms use row 4 (l / 16) + r).
//
// Operands are staged through LDS, 16 k-values per stage, as interleaved
// complex values (one 16-byte LDS access moves both parts).  The layout
// follows the operand's unit-stride dimension, so that the global loads are
// coalesced and neither the LDS writes nor the fragment reads (16 rows or
// columns at one k per 16 lanes) conflict: [k][64] where the tile's rows are
// unit stride, [row][16] with k XOR-permuted by the row where k is.
//
// The fp64 matrix cores are the bound (64 cycles per MFMA and SIMD), so the
// staging only has to stay out of their way: two LDS buffers with one
// barrier per stage, global loads issued two stages ahead, and eight waves
// per tile so that a launch of one tile per compute unit still has two waves
// per SIMD.  Measured against four waves, one buffer, separate planes and
// loads one stage ahead: 32,768-shot site GEMM at bond 1024 42 -> 65
// TFLOP/s, 1024 x 1024 x 2048 Gram (256 tiles) 26 -> 51, 2048 x 1024 x 1024
// product (512 tiles) 56 -> 57, two-site contraction at bond 1024 46 -> 55;
// four waves with this staging: 53, 35, 53 and 50.  The library's complex
// product reaches 65 at 2048^3.
//
// Operands come from loader functors so that each caller can gather rows or
// columns in its own way (row-indirect shot vectors, pairs of column blocks,
// conjugated transposes) while keeping global loads coalesced along the
// operand's unit-stride dimension.
#pragma once

#include "common.h"

namespace rcs {

constexpr int GT_M = 64, GT_N = 64, GT_K = 16;
constexpr int GT_THREADS = 512;
constexpr int GT_WN = GT_THREADS / 128;     // waves along N
constexpr int GT_NT = GT_N / GT_WN / 16;    // 16-column blocks per wave
constexpr int GT_PER = GT_M * GT_K / GT_THREADS;
static_assert(GT_M == GT_N && GT_K == 16, "the LDS layouts assume 64 x 64 x 16 stages");

struct SmemC64 {
  double2 a[2][GT_M * GT_K];
  double2 b[2][GT_N * GT_K];
};

struct AccC64 {
  double4_t re[2][GT_NT];
  double4_t im[2][GT_NT];
};

__device__ inline void acc_zero(AccC64& a) {
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < GT_NT; ++j) {
      a.re[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
      a.im[i][j] = double4_t{0.0, 0.0, 0.0, 0.0};
    }
}

// First row and column of wave w's part of the tile.
__device__ inline int wave_m(int w) { return (w & 1) * 32; }
__device__ inline int wave_n(int w) { return (w >> 1) * (16 * GT_NT); }

// LDS unit of tile row (or column) x at stage k.
template <bool KFAST>
__device__ inline int lds_unit(int x, int k) {
  if (KFAST) return x * 16 + (k ^ (x & 15));
  return k * 64 + x;
}

// Multiply the staged 64x16 A tile by the 16x64 B tile into the wave's part.
template <bool AK, bool BK>
__device__ inline void mma_stage(const double2* sa, const double2* sb, AccC64& acc, int wm, int wn, int lane) {
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < GT_K; kk += 4) {
    const int k = kk + lk;
    double2 a[2], b[GT_NT];
#pragma unroll
    for (int t = 0; t < 2; ++t) a[t] = sa[lds_unit<AK>(wm + t * 16 + lr, k)];
#pragma unroll
    for (int t = 0; t < GT_NT; ++t) b[t] = sb[lds_unit<BK>(wn + t * 16 + lr, k)];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int nt = 0; nt < GT_NT; ++nt) {
        acc.re[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt].x, b[nt].x, acc.re[mt][nt], 0, 0, 0);
        acc.im[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt].x, b[nt].y, acc.im[mt][nt], 0, 0, 0);
      }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int nt = 0; nt < GT_NT; ++nt) {
        acc.re[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[mt].y, b[nt].y, acc.re[mt][nt], 0, 0, 0);
        acc.im[mt][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[mt].y, b[nt].x, acc.im[mt][nt], 0, 0, 0);
      }
  }
}

// Output row (within a 16x16 block) of result register r in lane `lane`.
__device__ inline int f64_row(int lane, int r) { return (lane >> 4) + 4 * r; }

// Generic operand loader: element functor f(x, k) -> double2 for rows (or
// columns) x of the tile (absolute indices), with X x K bounds.  KFAST
// selects which index consecutive threads walk (the operand's unit-stride
// dimension).  fetch() reads a stage into registers, commit() writes them to
// LDS, so that the main loop can have the next stage's loads in flight
// during the current stage's matrix-core work.
template <class F, bool KFAST_>
struct LoadOp {
  static constexpr bool KFAST = KFAST_;
  F f;
  int x0, X, K;
  __device__ static inline void index(int j, int tid, int& x, int& k) {
    const int e = tid + j * GT_THREADS;
    if (KFAST) {
      k = e % GT_K;
      x = e / GT_K;
    } else {
      x = e % GT_M;
      k = e / GT_M;
    }
  }
  __device__ inline void fetch(double2 (&r)[GT_PER], int k0, int tid) const {
    if (x0 + GT_M <= X && k0 + GT_K <= K) {
#pragma unroll
      for (int j = 0; j < GT_PER; ++j) {
        int x, k;
        index(j, tid, x, k);
        r[j] = f(x0 + x, k0 + k);
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < GT_PER; ++j) {
      int x, k;
      index(j, tid, x, k);
      r[j] = (x0 + x < X && k0 + k < K) ? f(x0 + x, k0 + k) : make_double2(0.0, 0.0);
    }
  }
  __device__ inline void commit(double2* s, const double2 (&r)[GT_PER], int tid) const {
#pragma unroll
    for (int j = 0; j < GT_PER; ++j) {
      int x, k;
      index(j, tid, x, k);
      s[lds_unit<KFAST>(x, k)] = r[j];
    }
  }
};

// A operand f(m, k), M x K; KFAST: k is the unit-stride index.
template <class F, bool KFAST>
struct LoadA : LoadOp<F, KFAST> {
  __device__ LoadA(const F& f, int m0, int M, int K) : LoadOp<F, KFAST>{f, m0, M, K} {}
};

// B operand f(k, n), K x N; NFAST: n is the unit-stride index.
template <class F>
struct SwapArgs {
  F f;
  __device__ inline double2 operator()(int n, int k) const { return f(k, n); }
};
template <class F, bool NFAST>
struct LoadB : LoadOp<SwapArgs<F>, !NFAST> {
  __device__ LoadB(const F& f, int n0, int K, int N) : LoadOp<SwapArgs<F>, !NFAST>{SwapArgs<F>{f}, n0, N, K} {}
};

// K loop: the loads of stage s + 2 are issued before the matrix cores work
// on stage s; stage s + 1 goes from registers to the other LDS buffer after
// that work, so one barrier per stage orders both the new buffer's writes and
// the old one's reads.
template <class LA, class LB>
__device__ inline void cgemm_mainloop(const LA& la, const LB& lb, int K, SmemC64& s, AccC64& acc) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = wave_m(w), wn = wave_n(w);
  if (K <= 0) return;
  double2 ra[2][GT_PER], rb[2][GT_PER];
  la.fetch(ra[0], 0, tid);
  lb.fetch(rb[0], 0, tid);
  if (GT_K < K) {
    la.fetch(ra[1], GT_K, tid);
    lb.fetch(rb[1], GT_K, tid);
  }
  la.commit(s.a[0], ra[0], tid);
  lb.commit(s.b[0], rb[0], tid);
  __syncthreads();
  for (int k0 = 0; k0 < K; k0 += 2 * GT_K) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + h * GT_K;
      if (k >= K) return;
      if (k + 2 * GT_K < K) {
        la.fetch(ra[h], k + 2 * GT_K, tid);
        lb.fetch(rb[h], k + 2 * GT_K, tid);
      }
      mma_stage<LA::KFAST, LB::KFAST>(s.a[h], s.b[h], acc, wm, wn, lane);
      if (k + GT_K < K) {
        la.commit(s.a[h ^ 1], ra[h ^ 1], tid);
        lb.commit(s.b[h ^ 1], rb[h ^ 1], tid);
        __syncthreads();
      }
    }
  }
}

// Visit each output element held by this thread: g(row_in_tile, col_in_tile,
// re, im).
template <class G>
__device__ inline void acc_foreach(const AccC64& acc, G g) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = wave_m(w), wn = wave_n(w);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < GT_NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int row = wm + mt * 16 + f64_row(lane, r);
        int col = wn + nt * 16 + (lane & 15);
        g(row, col, acc.re[mt][nt][r], acc.im[mt][nt][r]);
      }
}

}  // namespace rcs
