// Triangular preconditioner for the one-sided Jacobi SVD: the Gram matrix
// G = X^H X of the two-site matrix, its Cholesky factor G = R^H R (R upper
// triangular), and Y = R^H in the Jacobi layout.
//
// X = Q R for some orthonormal Q, so X and R share singular values and right
// singular vectors.  One-sided Jacobi on Y = R^H converges in far fewer
// sweeps than on X (Drmac & Veselic, "New fast and accurate Jacobi SVD
// algorithm", SIAM J. Matrix Anal. Appl. 29, 2008: the triangular factor is
// one QR-iteration step closer to diagonal), and it leaves Y J = U_Y S with
// U_Y the right singular vectors of X, so neither Q nor the accumulated
// rotations J are needed.  R comes from the Gram rather than a Householder
// QR, which costs relative accuracy below the Gram's rounding level
// (singular values under ~1e-6 of the largest); the caller accepts the
// result only where that level cannot change the truncation, and otherwise
// runs the Jacobi on X itself.
//
// The factorisation is blocked by 64 columns, right-looking:
//   panel kernel:  every workgroup factors the 64 x 64 diagonal block of G
//                  in LDS (redundantly); workgroup 0 stores R_jj in a
//                  separate array (the others are still reading G_jj), the
//                  others solve their 64-column tile of the block row,
//                  R_jt = R_jj^{-H} G_jt;
//   update kernel: G_tu -= R_jt^H R_ju for the upper tiles of the trailing
//                  matrix, on the matrix cores.
// G is stored column-major with ld = round_up(n, 64); the padding carries an
// identity diagonal so that the padded matrix factors as blockdiag(R, I).
#include <utility>

#include "chol.h"
#include "gemm_f64.h"
#include "prof.h"

namespace rcs {

constexpr int CB = 64;          // Cholesky block

// Products C = A^H B over long columns (A: K x M, B: K x N, column-major).
// Up to about a thousand columns there are too few 64 x 64 tiles to fill the
// chip (136 on and above the diagonal at 1024 columns, 36 at 512, for 256
// compute units), so a tile's K range is split, units write partial tiles, and
// a second launch sums each tile's in order; one unit per tile stores its
// result itself.  Upper: only tiles on and above the diagonal (M = N).
// Bound: the fp64 matrix cores.  Measured: Gram of 2048 x 1024 in 3 ranges 221
// us instead of 330 (whole tiles, both triangles 336); the 20-qubit build at
// bond 512, whose Grams have 36 tiles and fewer, 234 -> 221 ms.
constexpr int AHB_MIN_K = 128;     // rows of a unit, at least
// Units of a split product, at most (64 KB of partials each): the 136 tiles of
// the 2048 x 1024 Gram get three ranges and their QR takes 2.62 ms; at most 256
// units leave them whole and it takes 2.83, at most 1,024 change nothing.
constexpr int AHB_UNITS = 576;

// Tile t of a product: row-major over all tiles, or over the upper triangle.
__device__ inline void ahb_tile(int t, int nbn, int upper, int& tm, int& tn) {
  if (!upper) {
    tm = t / nbn;
    tn = t % nbn;
    return;
  }
  tm = 0;
  while (t >= nbn - tm) {
    t -= nbn - tm;
    ++tm;
  }
  tn = tm + t;
}
template <class Store>
__global__ __launch_bounds__(GT_THREADS) void k_ahb(const double2* A, int lda, const double2* B, int ldb, int K, int M,
                                                   int N, int nbn, int upper, int kper, double2* part, Store store) {
  __shared__ SmemC64 sm;
  int tm, tn;
  ahb_tile(blockIdx.x, nbn, upper, tm, tn);
  const int m0 = tm * GT_M, n0 = tn * GT_N, k0 = blockIdx.y * kper, kn = min(kper, K - k0);
  auto fa = [&](int m, int k) -> double2 {
    const double2 v = A[(int64_t)m * lda + k0 + k];
    return make_double2(v.x, -v.y);
  };
  auto fb = [&](int k, int n) -> double2 { return B[(int64_t)n * ldb + k0 + k]; };
  LoadA<decltype(fa), true> la{fa, m0, M, kn};
  LoadB<decltype(fb), false> lb{fb, n0, kn, N};
  AccC64 acc;
  acc_zero(acc);
  cgemm_mainloop(la, lb, kn, sm, acc);
  if (gridDim.y == 1) {
    acc_foreach(acc, [&](int r, int c, double re, double im) { store(m0 + r, n0 + c, make_double2(re, im)); });
    return;
  }
  double2* out = part + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * (GT_M * GT_N);
  acc_foreach(acc, [&](int r, int c, double re, double im) { out[r * GT_N + c] = make_double2(re, im); });
}
template <class Store>
__global__ void k_ahb_sum(const double2* part, int splits, int nbn, int upper, Store store) {
  int tm, tn;
  ahb_tile(blockIdx.x, nbn, upper, tm, tn);
  const int e = blockIdx.y * blockDim.x + threadIdx.x;
  const double2* p = part + (int64_t)blockIdx.x * (GT_M * GT_N) + e;
  double2 s = p[0];
  for (int q = 1; q < splits; ++q) {
    const double2 v = p[(int64_t)q * gridDim.x * (GT_M * GT_N)];
    s.x += v.x;
    s.y += v.y;
  }
  store(tm * GT_M + e / GT_N, tn * GT_N + e % GT_N, s);
}

struct StoreGram {   // G (column-major), the identity beyond n
  double2* G;
  int ldg, n;
  __device__ void operator()(int m, int c, double2 v) const {
    if (m >= n || c >= n) v = make_double2(m == c ? 1.0 : 0.0, 0.0);
    G[(int64_t)c * ldg + m] = v;
  }
};
struct StoreNs {     // H = (3 I - C) / 2 (row-major), both triangles
  double2* H;
  int k;
  __device__ void operator()(int m, int c, double2 v) const {
    if (m >= k || c >= k) return;
    const double2 h = make_double2((m == c ? 1.5 : 0.0) - 0.5 * v.x, -0.5 * v.y);
    H[(int64_t)m * k + c] = h;
    if (m / GT_M != c / GT_N) H[(int64_t)c * k + m] = make_double2(h.x, -h.y);
  }
};
struct StoreP {      // scale C at m pm + c pn
  double2* P;
  int M, N;
  int64_t pm, pn;
  double scale;
  __device__ void operator()(int m, int c, double2 v) const {
    if (m < M && c < N) P[m * pm + c * pn] = make_double2(v.x * scale, v.y * scale);
  }
};

static int ahb_tiles(int M, int N, bool upper) {
  const int nbm = ceil_div(M, GT_M), nbn = ceil_div(N, GT_N);
  return upper ? nbn * (nbn + 1) / 2 : nbm * nbn;
}
// The number of K ranges that leaves the fewest rounds of the chip, and 0.02 of
// one charged for each range's partials.  Whole QR calls: without the charge
// 1500 x 700 takes 1.78 ms instead of 1.53 (ranges that only pay for
// themselves), with 0.05 or 0.1 1024 x 300 takes 0.67 or 0.71 instead of 0.63
// (unsplit 1.00).  Long narrow products would take more ranges than this gives
// them (8192 x 256: 1.00 ms, without the charge 0.72).
static int ahb_splits(int tiles, int K) {
  int best = 1;
  double cost = 1e30;
  for (int s = 1; s == 1 || (s <= 16 && s * AHB_MIN_K <= K && s * tiles <= AHB_UNITS); ++s) {
    const double c = (double)ceil_div(tiles * s, 256) / s + 0.02 * s;
    if (c < cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}
template <class Store>
static void ahb(const double2* A, int lda, const double2* B, int ldb, int K, int M, int N, bool upper, double2* part,
         const Store& store, hipStream_t s) {
  const int nbn = ceil_div(N, GT_N), tiles = ahb_tiles(M, N, upper);
  const int kper = (int)round_up(ceil_div(K, ahb_splits(tiles, K)), GT_K), splits = ceil_div(K, kper);
  RCS_PROBED_LAUNCH(kKcFactor, k_ahb<Store>, dim3(tiles, splits), dim3(GT_THREADS), 0, s, A, lda, B, ldb, K, M, N, nbn,
                    upper ? 1 : 0, kper, part, store);
  HIP_LAUNCH_OK();
  if (splits == 1) return;
  RCS_PROBED_LAUNCH(kKcFactor, k_ahb_sum<Store>, dim3(tiles, GT_M * GT_N / 256), dim3(256), 0, s, part, splits, nbn,
                    upper ? 1 : 0, store);
  HIP_LAUNCH_OK();
}

size_t ahb_part_bytes(int M, int N, int K, bool upper) {
  const int tiles = ahb_tiles(M, N, upper), splits = ahb_splits(tiles, K);
  return splits > 1 ? (size_t)tiles * splits * GT_M * GT_N * sizeof(double2) : 0;
}
void ns_gram(const double2* Q, int ldq, int len, int k, double2* H, double2* part, hipStream_t s) {
  ahb(Q, ldq, Q, ldq, len, k, k, true, part, StoreNs{H, k}, s);
}
void project(const double2* Q, int ldq, const double2* X, int ldx, int len, int k, int cnt, double scale, double2* P,
             int64_t pm, int64_t pn, double2* part, hipStream_t s) {
  ahb(Q, ldq, X, ldx, len, k, cnt, false, part, StoreP{P, k, cnt, pm, pn, scale}, s);
}

// Panel jb: every workgroup factors the 64 x 64 diagonal block G_jj = R^H R in
// LDS, in four 16-wide steps; workgroup t >= 1 carries its 64-column tile of
// the block row along (R_jt = R^{-H} G_jt), workgroup 0 stores R_jj
// (column-major in Rd) and, when Ri is given, the diagonal block of R^{-1}.
// A step:
//   factor  one wave factors the 16 x 16 diagonal block in registers (a column
//           per lane: no barrier in the 16-step chain), R^{-H} with it;
//   solve   the other blocks of the block row, times the inverse, and
//   update  the rows below, both as 16 x 16 matrix-core products, one block
//           per wave.
// A pivot that is not positive and finite sets *flag.
//
// Bound: the chain of 64 pivots (sqrt, division and a shuffle each).  Two
// barriers per pivot and per substitution row, with every thread's terms read
// from LDS, took 112 us per panel; this form with four rows of a column per
// lane, handed around by shuffles, 39 us, and with whole columns 31 us.
constexpr int PANEL_THREADS = 512;
constexpr int PW = 16;                     // inner block
constexpr int PLD = CB + 1;

struct PanelLds {
  double2 T[CB][PLD];                      // diagonal block, then R_jj
  double2 A[CB][PLD];                      // tile of the block row (workgroup 0: R_jj^{-1})
  double2 W[CB / PW][PW][PW + 1];          // R^{-H} of R_jj's 16 x 16 diagonal blocks
};

// B[r][cc] = G[row0 + r][col0 + cc] (G column-major, ld ldg) for a 64 x 64
// block, a thread's eight loads in flight before its LDS stores.
__device__ inline void load_block64(const double2* G, int ldg, int row0, int col0, double2 (*B)[PLD]) {
  constexpr int PER = CB * CB / PANEL_THREADS;
  const int r = threadIdx.x & (CB - 1), q = threadIdx.x >> 6;
  double2 v[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) v[u] = G[(int64_t)(col0 + q + (PANEL_THREADS / CB) * u) * ldg + row0 + r];
#pragma unroll
  for (int u = 0; u < PER; ++u) B[r][q + (PANEL_THREADS / CB) * u] = v[u];
}

__device__ inline double2 shfl2(double2 v, int lane) { return make_double2(__shfl(v.x, lane), __shfl(v.y, lane)); }

// a -= conj(t_I) s, t_I from lane I of the 16-lane row.
template <int I>
__device__ __forceinline__ void eliminate(double2& a, const double2& t, const double2& s) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, -%2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, -%2, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, -%3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
      : "+v"(a.x), "+v"(a.y)
      : "v"(t.x), "v"(t.y), "v"(s.x), "v"(s.y), "n"(I));
}
template <int K, int... J>
__device__ __forceinline__ void pivot_row(double2 (&a)[PW], int c, bool& bad, std::integer_sequence<int, J...>) {
  const double2 t = shfl2(a[K], c);   // row K of G in every 16-lane row
  double d = __shfl(t.x, K);
  if (!(d > 0.0) || !(d < 1e300)) {
    d = 1.0;
    bad = true;
  }
  const double inv = rsqrt_fast(d);
  const double2 r = make_double2(a[K].x * inv, a[K].y * inv), s = make_double2(r.x * inv, r.y * inv);
  (eliminate<K + 1 + J>(a[K + 1 + J], t, s), ...);
  a[K] = r;
}
template <int... K>
__device__ __forceinline__ void pivot_rows(double2 (&a)[PW], int c, bool& bad, std::integer_sequence<int, K...>) {
  (pivot_row<K>(a, c, bad, std::make_integer_sequence<int, PW - 1 - K>{}), ...);
}

// One wave: R^H R = T[k0.., k0..] (16 x 16, upper triangle used), R into T and
// R^{-H} (zero above the diagonal) into W.  The elimination runs on [G | I]:
// the row operations that turn G into R turn I into R^{-H}.  A lane holds one
// of the 32 columns (the wave's upper half repeats the lower one), and a
// pivot's multipliers are broadcast by the FMAs that use them.
__device__ inline void factor16(double2 (*T)[PLD], int k0, double2 (*W)[PW + 1], int lane, int* flag) {
  const int c = lane & 15;
  const bool left = (lane & 16) == 0;   // a column of G, else of I
  double2 a[PW];
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    const double2 g = T[k0 + i][k0 + c];
    a[i] = left ? g : make_double2(i == c ? 1.0 : 0.0, 0.0);
  }
  bool bad = false;
  pivot_rows(a, c, bad, std::make_integer_sequence<int, PW>{});
  if (bad && lane == 0) atomicExch(flag, 1);
  if (lane >= 32) return;
#pragma unroll
  for (int i = 0; i < PW; ++i) {
    if (left) {
      if (c >= i) T[k0 + i][k0 + c] = c == i ? make_double2(a[i].x, 0.0) : a[i];
    } else {
      W[i][c] = c <= i ? a[i] : make_double2(0.0, 0.0);
    }
  }
}

// One wave: acc (16 x 16) = A^H B (HERM) or A B of 16 x 16 LDS blocks.
struct Acc16 {
  double4_t re, im;
};
template <bool HERM, int LDA, int LDB>
__device__ inline Acc16 mul16(const double2 (*A)[LDA], int ar, int ac, const double2 (*B)[LDB], int br, int bc,
                              int lane) {
  Acc16 c{double4_t{0, 0, 0, 0}, double4_t{0, 0, 0, 0}};
  const int m = lane & 15, kl = lane >> 4;
#pragma unroll
  for (int kk = 0; kk < PW; kk += 4) {
    const int k = kk + kl;
    double2 x = HERM ? A[ar + k][ac + m] : A[ar + m][ac + k];
    if (HERM) x.y = -x.y;
    const double2 y = B[br + k][bc + m];
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.x, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, y.y, c.im, 0, 0, 0);
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, y.y, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.x, c.im, 0, 0, 0);
  }
  return c;
}

__global__ __launch_bounds__(PANEL_THREADS) void k_chol_panel(double2* G, int ldg, int jb, int* flag, double2* Rd,
                                                              double2* Ri) {
  __shared__ PanelLds sm;
  constexpr int NB = CB / PW, NWAVE = PANEL_THREADS / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, c = threadIdx.x & (CB - 1), q = threadIdx.x >> 6;
  const int j0 = jb * CB, t0 = j0 + blockIdx.x * CB;
  const bool tile = blockIdx.x > 0;
  load_block64(G, ldg, j0, j0, sm.T);
  if (tile) load_block64(G, ldg, j0, t0, sm.A);
  __syncthreads();
  for (int kb = 0; kb < NB; ++kb) {
    const int k0 = kb * PW;
    if (w == 0) factor16(sm.T, k0, sm.W[kb], lane, flag);
    __syncthreads();
    // block row kb: T's blocks right of the diagonal, the tile's four
    const int nt = NB - 1 - kb, solves = nt + (tile ? NB : 0);
    for (int e = w; e < solves; e += NWAVE) {
      double2(*M)[PLD] = e < nt ? sm.T : sm.A;
      const int col = e < nt ? (kb + 1 + e) * PW : (e - nt) * PW;
      const Acc16 x = mul16<false>(sm.W[kb], 0, 0, M, k0, col, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) M[k0 + f64_row(lane, r)][col + (lane & 15)] = make_double2(x.re[r], x.im[r]);
    }
    __syncthreads();
    // rows below: upper blocks of T, all four columns of the tile
    const int ut = nt * (nt + 1) / 2, updates = ut + (tile ? nt * NB : 0);
    for (int e = w; e < updates; e += NWAVE) {
      int ti, col;
      double2(*M)[PLD] = sm.T;
      if (e < ut) {
        int p = e;
        ti = 0;
        while (p >= nt - ti) {
          p -= nt - ti;
          ++ti;
        }
        col = (kb + 1 + ti + p) * PW;
      } else {
        ti = (e - ut) / NB;
        col = ((e - ut) % NB) * PW;
        M = sm.A;
      }
      const int row = (kb + 1 + ti) * PW;
      const Acc16 x = mul16<true>(sm.T, k0, row, M, k0, col, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double2& v = M[row + f64_row(lane, r)][col + (lane & 15)];
        v = make_double2(v.x - x.re[r], v.y - x.im[r]);
      }
    }
    __syncthreads();
  }
  if (tile) {
    for (int cc = q; cc < CB; cc += NWAVE) G[(int64_t)(t0 + cc) * ldg + j0 + c] = sm.A[c][cc];
    return;
  }
  double2* rd = Rd + (int64_t)jb * CB * CB;
  for (int cc = q; cc < CB; cc += NWAVE) rd[cc * CB + c] = c <= cc ? sm.T[c][cc] : make_double2(0.0, 0.0);
  if (!Ri) return;
  // R_jj^{-1} from its 16 x 16 diagonal blocks: the block diagonals above the
  // main one in turn, X_ij = -R_ii^{-1} sum_{i < l <= j} R_il X_lj
  for (int e = threadIdx.x; e < CB * CB; e += PANEL_THREADS) {
    const int i = e / CB, j = e % CB;
    const double2 v = sm.W[i / PW][j % PW][i % PW];
    sm.A[i][j] = i / PW == j / PW ? make_double2(v.x, -v.y) : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int dgn = 1; dgn < NB; ++dgn) {
    const int i = w, j = w + dgn;
    const bool mine = j < NB;
    if (mine) {
      double4_t re{0, 0, 0, 0}, im{0, 0, 0, 0};
      for (int l = i + 1; l <= j; ++l) {
        const Acc16 x = mul16<false>(sm.T, i * PW, l * PW, sm.A, l * PW, j * PW, lane);
        re += x.re;
        im += x.im;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.A[i * PW + f64_row(lane, r)][j * PW + (lane & 15)] = make_double2(re[r], im[r]);
    }
    __syncthreads();
    Acc16 y;
    if (mine) y = mul16<true>(sm.W[i], 0, 0, sm.A, i * PW, j * PW, lane);
    __syncthreads();
    if (mine) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sm.A[i * PW + f64_row(lane, r)][j * PW + (lane & 15)] = make_double2(-y.re[r], -y.im[r]);
    }
    __syncthreads();
  }
  for (int cc = q; cc < CB; cc += NWAVE)
    Ri[(int64_t)(j0 + cc) * ldg + j0 + c] = sm.A[c][cc];
}

// Trailing update after panel jb: tile (ti, tj), jb < ti <= tj < nb:
// G_{ti,tj} -= R_{jb,ti}^H R_{jb,tj}.  blockIdx.x enumerates the pairs.
__global__ __launch_bounds__(GT_THREADS) void k_chol_update(double2* G, int ldg, int nb, int jb) {
  __shared__ SmemC64 sm;
  const int T = nb - jb - 1;
  // pair index -> (ti, tj) with ti <= tj, row-major over the upper triangle
  int p = blockIdx.x, ti = 0;
  while (p >= T - ti) {
    p -= T - ti;
    ++ti;
  }
  const int tj = ti + p;
  const int r0 = (jb + 1 + ti) * CB, c0 = (jb + 1 + tj) * CB, k0 = jb * CB;
  auto fa = [&](int m, int kk) -> double2 {
    const double2 v = G[(int64_t)(r0 + m) * ldg + k0 + kk];
    return make_double2(v.x, -v.y);
  };
  auto fb = [&](int kk, int n) -> double2 { return G[(int64_t)(c0 + n) * ldg + k0 + kk]; };
  LoadA<decltype(fa), true> la{fa, 0, CB, CB};
  LoadB<decltype(fb), false> lb{fb, 0, CB, CB};
  AccC64 acc;
  acc_zero(acc);
  cgemm_mainloop(la, lb, CB, sm, acc);
  acc_foreach(acc, [&](int r, int c, double re, double im) {
    double2* g = G + (int64_t)(c0 + c) * ldg + r0 + r;
    *g = make_double2(g->x - re, g->y - im);
  });
}

// Y (ldy x ncols, column-major) = R^H in the leading n x n block, zero
// elsewhere; R's diagonal blocks are in Rd (64 x 64 each, column-major), its
// off-diagonal blocks in the upper triangle of G.
__global__ void k_chol_to_y(const double2* G, int ldg, const double2* Rd, int n, double2* Y, int ldy, int ncols) {
  const int64_t tot = (int64_t)ldy * ncols;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < tot;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int i = (int)(e % ldy), j = (int)(e / ldy);
    double2 v = make_double2(0.0, 0.0);
    if (i < n && j < n && i >= j) {
      // R[j][i], row j, column i
      const double2 r = (i / CB == j / CB) ? Rd[(int64_t)(j / CB) * CB * CB + (i % CB) * CB + (j % CB)]
                                           : G[(int64_t)i * ldg + j];
      v = make_double2(r.x, -r.y);
    }
    Y[e] = v;
  }
}

// Gram and blocked Cholesky (R's off-diagonal blocks in G, diagonal blocks
// in Rd, diagonal blocks of R^{-1} in Ri when Ri is not null).
static void gram_cholesky(const double2* X, int ldx, int len, int n, double2* G, int ldg, double2* Rd, double2* Ri,
                          int* flag_dev, double2* part, hipStream_t s) {
  RCS_REQUIRE(ldg % CB == 0 && ldg >= n, "Gram leading dimension must be a multiple of 64");
  const int nb = ldg / CB;
  ahb(X, ldx, X, ldx, len, n, n, true, part, StoreGram{G, ldg, n}, s);
  for (int jb = 0; jb < nb; ++jb) {
    RCS_PROBED_LAUNCH(kKcFactor, k_chol_panel, dim3(nb - jb), dim3(PANEL_THREADS), 0, s, G, ldg, jb, flag_dev, Rd, Ri);
    HIP_LAUNCH_OK();
    const int T = nb - jb - 1;
    if (T > 0) {
      RCS_PROBED_LAUNCH(kKcFactor, k_chol_update, dim3(T * (T + 1) / 2), dim3(GT_THREADS), 0, s, G, ldg, nb, jb);
      HIP_LAUNCH_OK();
    }
  }
}

void chol_precondition(const double2* X, int ldx, int len, int n, double2* G, int ldg, double2* Rd, double2* Y,
                       int ldy, int ycols, int* flag_dev, double2* part, hipStream_t s) {
  gram_cholesky(X, ldx, len, n, G, ldg, Rd, nullptr, flag_dev, part, s);
  const int64_t tot = (int64_t)ldy * ycols;
  RCS_PROBED_LAUNCH(kKcFactor, k_chol_to_y, dim3((unsigned)std::min<int64_t>((tot + 255) / 256, 65535)), dim3(256), 0, s, G,
                     ldg, Rd, n, Y, ldy, ycols);
  HIP_LAUNCH_OK();
}

// Batched column-major complex GEMM on sub-blocks: for batch z,
// D_z = alpha A_z B_z with A_z = A + z sa (M x K, ld lda), B_z = B + z sb
// (K x N, ld ldb), D_z = D + z sd (M x N, ld ldd), overwritten.  kUpperA /
// kUpperB: that operand is upper triangular, and the K range it leaves zero in
// a tile is not gone through (half of the work).
enum { kUpperA, kUpperB };
__global__ __launch_bounds__(GT_THREADS) void k_cgemm_cm(const double2* A, int lda, int64_t sa, const double2* B,
                                                        int ldb, int64_t sb, double2* D, int ldd, int64_t sd, int M,
                                                        int N, int K, double alpha, int upper) {
  __shared__ SmemC64 sm;
  const int64_t z = blockIdx.z;
  const double2* a = A + z * sa;
  const double2* b = B + z * sb;
  double2* d = D + z * sd;
  // a triangular B's columns from the longest in the launch's first half and
  // from the shortest in its second, so that a compute unit with one tile of
  // each has about the average work
  const bool flip = upper == kUpperB && 2 * blockIdx.y < gridDim.y;
  const int m0 = blockIdx.y * GT_M, n0 = (flip ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x) * GT_N;
  const int k0 = upper == kUpperA ? m0 : 0, kn = (upper == kUpperB ? min(K, n0 + GT_N) : K) - k0;
  auto fa = [&](int m, int k) -> double2 { return a[(int64_t)(k0 + k) * lda + m]; };
  auto fb = [&](int k, int n) -> double2 { return b[(int64_t)n * ldb + k0 + k]; };
  LoadA<decltype(fa), false> la{fa, m0, M, kn};
  LoadB<decltype(fb), false> lb{fb, n0, kn, N};
  AccC64 acc;
  acc_zero(acc);
  cgemm_mainloop(la, lb, kn, sm, acc);
  acc_foreach(acc, [&](int r, int c, double re, double im) {
    const int m = m0 + r, n = n0 + c;
    if (m < M && n < N) d[(int64_t)n * ldd + m] = make_double2(alpha * re, alpha * im);
  });
}

static void cgemm_cm(const double2* A, int lda, int64_t sa, const double2* B, int ldb, int64_t sb, double2* D,
                     int ldd, int64_t sd, int M, int N, int K, double alpha, int batch, int upper, hipStream_t s) {
  if (batch <= 0 || M <= 0 || N <= 0) return;
  RCS_PROBED_LAUNCH(kKcFactor, k_cgemm_cm, dim3(ceil_div(N, GT_N), ceil_div(M, GT_M), batch), dim3(GT_THREADS), 0, s, A, lda,
                     sa, B, ldb, sb, D, ldd, sd, M, N, K, alpha, upper);
  HIP_LAUNCH_OK();
}

// R^{-1} (upper, ld ldg, lower part zero) from its 64 x 64 diagonal blocks
// (already in Ri) by recursive doubling: for blocks [A | C] of the leading
// diagonal, R^{-1}_{AC} = -R^{-1}_{AA} R_{AC} R^{-1}_{CC}, all pairs of a
// level at once (two GEMM launches per level; T is an ldg x ldg scratch).
static void triangular_inverse(const double2* G, int ldg, double2* Ri, double2* T, hipStream_t s) {
  for (int h = CB; h < ldg; h *= 2) {
    const int full = ldg / (2 * h);              // pairs with |C| = h
    const int tail0 = full * 2 * h;              // a last pair with |C| < h
    const int64_t stride = (int64_t)2 * h * ldg + 2 * h;
    // T_AC = R_AC R^{-1}_CC, then Ri_AC = -R^{-1}_AA T_AC
    cgemm_cm(G + (int64_t)h * ldg, ldg, stride, Ri + (int64_t)h * ldg + h, ldg, stride, T + (int64_t)h * ldg, ldg,
             stride, h, h, h, 1.0, full, kUpperB, s);
    cgemm_cm(Ri, ldg, stride, T + (int64_t)h * ldg, ldg, stride, Ri + (int64_t)h * ldg, ldg, stride, h, h, h, -1.0,
             full, kUpperA, s);
    const int hc = ldg - tail0 - h;
    if (hc > 0) {
      const int64_t a0 = (int64_t)tail0 * ldg + tail0, c0 = (int64_t)(tail0 + h) * ldg + (tail0 + h);
      const int64_t ac = (int64_t)(tail0 + h) * ldg + tail0;
      cgemm_cm(G + ac, ldg, 0, Ri + c0, ldg, 0, T + ac, ldg, 0, h, hc, hc, 1.0, 1, kUpperB, s);
      cgemm_cm(Ri + a0, ldg, 0, T + ac, ldg, 0, Ri + ac, ldg, 0, h, hc, h, -1.0, 1, kUpperA, s);
    }
  }
}

void cholqr(const double2* X, int ldx, int len, int n, double2* G, int ldg, double2* Rd, double2* Ri, double2* T,
            double2* Q, int ldq, int* flag_dev, double2* part, hipStream_t s) {
  HIP_OK(hipMemsetAsync(Ri, 0, (size_t)ldg * ldg * sizeof(double2), s));
  gram_cholesky(X, ldx, len, n, G, ldg, Rd, Ri, flag_dev, part, s);
  triangular_inverse(G, ldg, Ri, T, s);
  cgemm_cm(X, ldx, 0, Ri, ldg, 0, Q, ldq, 0, len, n, n, 1.0, 1, kUpperB, s);
}

// *dev = max over entries of |H - I| (H k x k, row-major); *dev must be 0
// beforehand.  Non-negative doubles order like their bit patterns, so the
// workgroups combine with an integer atomic max.
__global__ void k_max_dev_identity(const double2* H, int k, double* dev) {
  __shared__ double red[256];
  double m = 0.0;
  const int64_t tot = (int64_t)k * k;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < tot; e += (int64_t)gridDim.x * 256) {
    const int r = (int)(e / k), c = (int)(e % k);
    const double2 h = H[e];
    const double re = h.x - (r == c ? 1.0 : 0.0);
    m = fmax(m, fmax(fabs(re), fabs(h.y)));
    if (!(h.x == h.x) || !(h.y == h.y)) m = 1e300;
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int h2 = 128; h2 > 0; h2 >>= 1) {
    if ((int)threadIdx.x < h2) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + h2]);
    __syncthreads();
  }
  if (threadIdx.x == 0)
    atomicMax(reinterpret_cast<unsigned long long*>(dev), (unsigned long long)__double_as_longlong(red[0]));
}

void max_dev_identity(const double2* H, int k, double* dev, hipStream_t s) {
  HIP_OK(hipMemsetAsync(dev, 0, sizeof(double), s));
  const int64_t tot = (int64_t)k * k;
  const int blocks = (int)std::min<int64_t>(1024, (tot + 255) / 256);
  RCS_PROBED_LAUNCH(kKcFactor, k_max_dev_identity, dim3(std::max(blocks, 1)), dim3(256), 0, s, H, k, dev);
  HIP_LAUNCH_OK();
}

// P (k x len, row-major) = scale * (X U)^H with X len x n (ld ldx) and U
// n x k (ld ldu): P[j][r] = scale * sum_i conj(U[i][j]) conj(X[r][i]).
__global__ __launch_bounds__(GT_THREADS) void k_project_rows(const double2* U, int ldu, const double2* X, int ldx,
                                                            int len, int n, int k, double scale, double2* P) {
  __shared__ SmemC64 sm;
  const int m0 = blockIdx.y * GT_M, n0 = blockIdx.x * GT_N;
  auto fa = [&](int j, int i) -> double2 {
    const double2 v = U[(int64_t)j * ldu + i];
    return make_double2(v.x, -v.y);
  };
  auto fb = [&](int i, int r) -> double2 {
    const double2 v = X[(int64_t)i * ldx + r];
    return make_double2(v.x, -v.y);
  };
  LoadA<decltype(fa), true> la{fa, m0, k, n};
  LoadB<decltype(fb), true> lb{fb, n0, n, len};
  AccC64 acc;
  acc_zero(acc);
  cgemm_mainloop(la, lb, n, sm, acc);
  acc_foreach(acc, [&](int r, int c, double re, double im) {
    const int j = m0 + r, col = n0 + c;
    if (j < k && col < len) P[(int64_t)j * len + col] = make_double2(re * scale, im * scale);
  });
}

void project_rows(const double2* U, int ldu, const double2* X, int ldx, int len, int n, int k, double scale,
                  double2* P, hipStream_t s) {
  RCS_PROBED_LAUNCH(kKcFactor, k_project_rows, dim3(ceil_div(len, GT_N), ceil_div(k, GT_M)), dim3(GT_THREADS), 0, s, U, ldu,
                     X, ldx, len, n, k, scale, P);
  HIP_LAUNCH_OK();
}

// out[j*ld + order[i]] = in[j*ld + i] for i < n, j < k: rows back to the
// caller's column order.
__global__ void k_unpermute_rows(const double2* in, int ld, int n, int k, const int* order, double2* out) {
  const int j = blockIdx.y;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    out[(int64_t)j * ld + order[i]] = in[(int64_t)j * ld + i];
}

void unpermute_rows(const double2* in, int ld, int n, int k, const int* order, double2* out, hipStream_t s) {
  RCS_PROBED_LAUNCH(kKcFactor, k_unpermute_rows, dim3(ceil_div(n, 256), k), dim3(256), 0, s, in, ld, n, k, order, out);
  HIP_LAUNCH_OK();
}

}  // namespace rcs
