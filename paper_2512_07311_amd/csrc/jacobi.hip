// One-sided block Jacobi SVD (Hestenes method, block variant with a
// Gram-matrix inner eigensolver), in fp64 or fp32 (complex128 / complex64
// data, the matching matrix-core products; R below is the real type and u
// its unit roundoff).
//
// X (len x cnt, complex, column-major, leading dimension ldx, zero padded to
// nbp*16 columns) is rotated from the right by unitary 32x32 block rotations
// until every pair of columns is orthogonal to the relative tolerance
// tol = 16 u sqrt(len) (fresh Grams keep relative accuracy; the margin over
// the rounding noise of a length-len inner product keeps noise from
// re-triggering rotations among millions of pairs), ignoring columns
// below the noise level delta ||X||_F; the columns are then
// sigma_j u_j.  Per sweep the nbp column blocks (16 columns each) meet
// pairwise in round-robin order: nbp-1 rounds of nbp/2 disjoint pairs.  A
// round is two launches:
//   gram   : G_p = Y_p^H Y_p, Y_p = [X_bi | X_bj], as partial Grams over row
//            chunks (MFMA in R; waves reduce in fixed order);
//   rotate : every (pair, chunk) workgroup sums the partial Grams in fixed
//            order, diagonalises the 32x32 Hermitian G_p in LDS by cyclic
//            two-sided Jacobi (all workgroups of a pair compute the same
//            rotations), and applies them to its own rows: in fp64 each
//            rotation directly, to rows held in registers; in fp32 and for
//            32-column blocks as the product Y_p V_p on the matrix cores.
// A pair whose two blocks were not rotated since the pair last met is
// skipped (it is still orthogonal), so late sweeps cost almost nothing.  A
// sweep that rotates nothing ends the iteration, and so does a sweep whose
// meetings all entered with squared cosines below tol / 100 (the rotate
// pass raises a flag otherwise): at that point convergence is quadratic and
// the next sweep would rotate nothing.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "gemm_f64.h"
#include "jacobi.h"
#include "jacobi_dev.h"
#include "prof.h"

namespace rcs {

constexpr int TR = 16;        // rows per wave tile (four 4-row MFMA k steps)

__device__ inline int rr_block(int slot, int round, int nbp) {
  return slot == 0 ? 0 : ((slot - 1 + round) % (nbp - 1)) + 1;
}

template <typename R>
struct JacArgs {
  typename JT<R>::C* x;
  int ldx, len, nbp, round, rows_per_chunk, n_chunks;   // rotate chunks
  int rows_per_gchunk, n_gchunks;                      // Gram chunks
  typename JT<R>::C* part;   // [pair][chunk][JP][JP], cross rounds of the row-resident pass: [pair][chunk][16][16]
  int* rot_prev;      // [nbp] block rotated during the previous sweep
  int* rot_cur;       // [nbp] block rotated during this sweep
  int* rot_count;
  int* big_cos;       // set when a meeting entered with |g_ij|^2 > qtol g_ii g_jj
  R qtol;             // squared-cosine level below which the next sweep would rotate nothing
  R tol;              // relative orthogonality tolerance
  R neg2;             // squared column norm below which a column counts as zero
  int max_inner;      // inner two-sided sweeps per pair meeting
  typename JT<R>::C* bg;     // row-resident pass: [2][block][16][16], the blocks' own Grams
};

template <typename R>
__device__ inline bool pair_skipped(const JacArgs<R>& a, int bi, int bj) {
  return a.rot_prev[bi] == 0 && a.rot_prev[bj] == 0 && a.rot_cur[bi] == 0 && a.rot_cur[bj] == 0;
}

template <int JP>
__device__ inline int pair_col(int c, int bi, int bj) {
  return c < JP / 2 ? bi * (JP / 2) + c : bj * (JP / 2) + (c - JP / 2);
}

// Lane's element of every 16-column block of Y_p at one row (zero past
// rend).  The lane's column within a block is lane % 16, so a load
// instruction covers 16 columns x 4 consecutive rows.
template <int JP, typename C>
__device__ inline void load_row(const C* x, int ldx, int bi, int bj, int row, int rend, C (&v)[JP / 16], int lane) {
#pragma unroll
  for (int cb = 0; cb < JP / 16; ++cb) {
    const int col = pair_col<JP>(cb * 16 + (lane & 15), bi, bj);
    v[cb] = row < rend ? x[(int64_t)col * ldx + row] : C(0, 0);
  }
}

// Partial Grams.  Waves split the chunk's rows (16-row tiles, interleaved)
// and each accumulates the NB(NB+1)/2 upper 16x16 blocks of Y^H Y on the
// matrix cores straight from registers; the waves are then summed through LDS
// in a fixed order (waves 4-7, if any, into 0-3, then ((w3 + w2) + w1) + w0).
//
// Waves per workgroup: four, each with its own 16-row tile of a 64-row chunk,
// are the fastest launch of a small matrix (5.6 us against 7.2 with eight at
// 512 x 512).  But every rotate workgroup of a pair reads all of the pair's
// partials (16 KB each), and from about 768 rows that traffic costs more than
// the launch: in fp64, eight waves on 128-row chunks make a whole round 27.7
// us against 29.6 at 1024 x 1024 and 56.4 against 58.4 at 2048 x 2048
// (sixteen waves: 30.8 and 59.8).  The fp32 pass keeps four waves: its
// partials are half the size, and its singular values depend on the
// summation order at the 1e-4 level of its drift.
//
// CROSS: only the product of the two blocks with each other; the rotate pass
// has their own Grams from the blocks' previous meeting.
template <int JP, int NW, typename R, bool CROSS = false>
__global__ __launch_bounds__(64 * NW) void k_jac_gram(JacArgs<R> a) {
  using T = JT<R>;
  using C = typename T::C;
  using V4 = typename T::V4;
  constexpr int NB = JP / 16, NU = CROSS ? 1 : NB * (NB + 1) / 2;
  static_assert(NW == 4 || NW == 8, "the reduction below");
  static_assert(!CROSS || JP == 32, "two 16-column blocks");
  __shared__ R red[NW == 8 ? 4 : 1][NU * 8][64];
  const int p = blockIdx.x, chunk = blockIdx.y;
  const int bi = rr_block(p, a.round, a.nbp), bj = rr_block(a.nbp - 1 - p, a.round, a.nbp);
  if (pair_skipped(a, bi, bj)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int rbeg = chunk * a.rows_per_gchunk;
  const int rend = min(a.len, rbeg + a.rows_per_gchunk);
  const int ntiles = (rend - rbeg + TR - 1) / TR;
  V4 gr[NU], gi[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    gr[u] = V4{0, 0, 0, 0};
    gi[u] = V4{0, 0, 0, 0};
  }
  C cur[4][NB], nxt[4][NB];
  const int rsub = lane >> 4;
  if (w < ntiles) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      load_row<JP>(a.x, a.ldx, bi, bj, rbeg + w * TR + 4 * ks + rsub, rend, cur[ks], lane);
  }
  for (int t = w; t < ntiles; t += NW) {
    if (t + NW < ntiles) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        load_row<JP>(a.x, a.ldx, bi, bj, rbeg + (t + NW) * TR + 4 * ks + rsub, rend, nxt[ks], lane);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      auto product = [&](int u, const C& ym, const C& yn) {
        gr[u] = T::mma(ym.x, yn.x, gr[u]);
        gr[u] = T::mma(ym.y, yn.y, gr[u]);
        gi[u] = T::mma(ym.x, yn.y, gi[u]);
        gi[u] = T::mma(-ym.y, yn.x, gi[u]);
      };
      if constexpr (CROSS) {
        product(0, cur[ks][0], cur[ks][1]);
      } else {
        int u = 0;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb)
#pragma unroll
          for (int nb = mb; nb < NB; ++nb, ++u) product(u, cur[ks][mb], cur[ks][nb]);
      }
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) cur[ks][cb] = nxt[ks][cb];
  }
  if constexpr (NW == 8) {
    if (w >= 4) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          red[w - 4][u * 8 + r][lane] = gr[u][r];
          red[w - 4][u * 8 + 4 + r][lane] = gi[u][r];
        }
    }
    __syncthreads();
    if (w < 4) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gr[u][r] += red[w][u * 8 + r][lane];
          gi[u][r] += red[w][u * 8 + 4 + r][lane];
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int src = 3; src >= 1; --src) {
    if (w == src) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          R vr = gr[u][r], vi = gi[u][r];
          if (src < 3) {
            vr += red[0][u * 8 + r][lane];
            vi += red[0][u * 8 + 4 + r][lane];
          }
          red[0][u * 8 + r][lane] = vr;
          red[0][u * 8 + 4 + r][lane] = vi;
        }
    }
    __syncthreads();
  }
  if (w != 0) return;
  if constexpr (CROSS) {
    C* part = a.part + ((int64_t)p * a.n_gchunks + chunk) * 256;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      part[T::orow(lane, r) * 16 + (lane & 15)] = T::mk(gr[0][r] + red[0][r][lane], gi[0][r] + red[0][4 + r][lane]);
    return;
  }
  C* part = a.part + ((int64_t)p * a.n_gchunks + chunk) * JP * JP;
  int u = 0;
#pragma unroll
  for (int mb = 0; mb < NB; ++mb)
#pragma unroll
    for (int nb = mb; nb < NB; ++nb, ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const R vr = gr[u][r] + red[0][u * 8 + r][lane];
        const R vi = gi[u][r] + red[0][u * 8 + 4 + r][lane];
        const int row = mb * 16 + T::orow(lane, r), col = nb * 16 + (lane & 15);
        part[row * JP + col] = T::mk(vr, vi);
        if (mb != nb) part[col * JP + row] = T::mk(vr, -vi);
      }
}

// Members (i < j) of pair q in round-robin round `round` of JP columns, and
// the pair that column c belongs to in that round.
template <int JP>
__device__ inline void rr_pair(int q, int round, int& i, int& j) {
  const int u = q == 0 ? 0 : ((q - 1 + round) % (JP - 1)) + 1;
  const int v = ((JP - 2 - q + round) % (JP - 1)) + 1;
  i = min(u, v);
  j = max(u, v);
}
template <int JP>
__device__ inline int rr_pair_of(int c, int round) {
  const int slot = c == 0 ? 0 : ((c - 1 - round + 2 * (JP - 1)) % (JP - 1)) + 1;
  return min(slot, JP - 1 - slot);
}

constexpr int ROT_THREADS = 512;

// Y_p <- Y_p V_p for this chunk's rows on the matrix cores (all ROT_THREADS).
template <int JP, typename R, int LDV>
__device__ inline void rotate_rows_by(const JacArgs<R>& a, const typename JT<R>::C (*V)[LDV], int bi, int bj,
                                      int chunk) {
  using T = JT<R>;
  using C = typename T::C;
  using V4 = typename T::V4;
  constexpr int NB = JP / 16;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // waves take 16-row tiles; A operand straight from global
  // (16 consecutive rows of one column per 16 lanes), B = V from LDS.
  const int rbeg = chunk * a.rows_per_chunk;
  const int rend = min(a.len, rbeg + a.rows_per_chunk);
  const int ntiles = (rend - rbeg + TR - 1) / TR;
  constexpr int KS = JP / 4, NW = ROT_THREADS / 64;
  C cur[KS], nxt[KS];
  const int m = lane & 15, ksub = lane >> 4;
  auto load_tile_regs = [&](int tt, C (&v)[KS]) {
    const int row = rbeg + tt * TR + m;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int col = pair_col<JP>(4 * ks + ksub, bi, bj);
      v[ks] = row < rend ? a.x[(int64_t)col * a.ldx + row] : C(0, 0);
    }
  };
  if (w < ntiles) load_tile_regs(w, cur);
  for (int tt = w; tt < ntiles; tt += NW) {
    if (tt + NW < ntiles) load_tile_regs(tt + NW, nxt);
    V4 cr[NB], ci[NB];
#pragma unroll
    for (int nt = 0; nt < NB; ++nt) {
      cr[nt] = V4{0, 0, 0, 0};
      ci[nt] = V4{0, 0, 0, 0};
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const C y = cur[ks];
      const int k = 4 * ks + ksub;
#pragma unroll
      for (int nt = 0; nt < NB; ++nt) {
        const C v = V[k][nt * 16 + m];
        cr[nt] = T::mma(y.x, v.x, cr[nt]);
        cr[nt] = T::mma(-y.y, v.y, cr[nt]);
        ci[nt] = T::mma(y.x, v.y, ci[nt]);
        ci[nt] = T::mma(y.y, v.x, ci[nt]);
      }
    }
    const int row0 = rbeg + tt * TR;
#pragma unroll
    for (int nt = 0; nt < NB; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + T::orow(lane, r);
        const int col = nt * 16 + m;
        if (row < rend) a.x[(int64_t)pair_col<JP>(col, bi, bj) * a.ldx + row] = T::mk(cr[nt][r], ci[nt][r]);
      }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) cur[ks] = nxt[ks];
  }
  if (chunk == 0 && tid == 0) {
    a.rot_cur[bi] = 1;
    a.rot_cur[bj] = 1;
    atomicAdd(a.rot_count, 1);
  }
}

// Sum partial Grams (fixed order), diagonalise the JP x JP Hermitian G_p by
// cyclic two-sided Jacobi in LDS (every workgroup of a pair computes the
// same unitary V_p), and rotate this chunk's rows, Y_p <- Y_p V_p, on the
// matrix cores.
//
// Inner solve: a round applies JP/2 disjoint rotations at once.  JP/2 lanes
// compute the round's rotations into LDS; then waves 0-3 take the (JP/2)^2
// blocks G[pair a, pair b] <- J_a^H G[a, b] J_b and waves 4-7 the blocks
// V[rows of a, pair b] <- V J_b (one of each per SIMD, so their latencies
// overlap), all in place: each entry belongs to one job per round.  The
// diagonal and the next round's pair entries are handed on through small
// double-buffered arrays.  Used by 64-column pairs and, in fp32, by a sweep's
// first round; k_jac_rotate_cross has the other fp32 rounds.
template <int JP, typename R>
__global__ __launch_bounds__(ROT_THREADS) void k_jac_rotate(JacArgs<R> a) {
  using T = JT<R>;
  using C = typename T::C;
  using V4 = typename T::V4;
  constexpr int GS = JP + 1, NP = JP / 2, NB = JP / 16, JOBS = NP * NP / 256;
  static_assert(NP * NP % 256 == 0, "block jobs must tile a wave group");
  __shared__ C G[JP][GS];
  __shared__ C V[JP][GS];
  __shared__ R dd[2][JP];
  __shared__ C od[2][NP];
  __shared__ unsigned char tb_i[JP - 1][NP], tb_j[JP - 1][NP], tb_q[JP - 1][JP];
  __shared__ RotA<R> rp[NP];
  __shared__ int any_flag;
  __shared__ int big_lds;
  const int p = blockIdx.x, chunk = blockIdx.y;
  const int bi = rr_block(p, a.round, a.nbp), bj = rr_block(a.nbp - 1 - p, a.round, a.nbp);
  if (pair_skipped(a, bi, bj)) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const C* part = a.part + (int64_t)p * a.n_gchunks * JP * JP;
  for (int e = tid; e < JP * JP; e += ROT_THREADS) {
    // partials summed in chunk order; loads issued eight at a time
    C s(0, 0);
    for (int c0 = 0; c0 < a.n_gchunks; c0 += 8) {
      C t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        t[u] = c0 + u < a.n_gchunks ? part[(int64_t)(c0 + u) * JP * JP + e] : C(0, 0);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s.x += t[u].x;
        s.y += t[u].y;
      }
    }
    const int i = e / JP, j = e % JP;
    G[i][j] = s;
    V[i][j] = T::mk(i == j ? 1 : 0, 0);
  }
  if (tid == 0) {
    any_flag = 0;
    big_lds = 0;
  }
  // Inner schedule tables: members of pair q and the pair of column c, per
  // round.  The first outer round of a sweep runs the full round-robin over
  // all JP(JP-1)/2 column pairs (every block meets there, so every
  // intra-block pair is rotated once per sweep); the other outer rounds
  // rotate only the (JP/2)^2 cross pairs, column q of block bi against
  // column (q + t) mod JP/2 of block bj in round t.  Every column pair is
  // thus rotated at least once per sweep, as in cyclic Jacobi, at half the
  // inner rounds.
  const bool full = a.round == 0;
  const int n_in = full ? JP - 1 : NP;
  for (int e = tid; e < n_in * NP; e += ROT_THREADS) {
    const int rd = e / NP, q = e % NP;
    int i, j;
    if (full) {
      rr_pair<JP>(q, rd, i, j);
    } else {
      i = q;
      j = NP + (q + rd) % NP;
    }
    tb_i[rd][q] = (unsigned char)i;
    tb_j[rd][q] = (unsigned char)j;
  }
  for (int e = tid; e < n_in * JP; e += ROT_THREADS) {
    const int rd = e / JP, c = e % JP;
    tb_q[rd][c] = (unsigned char)(full ? rr_pair_of<JP>(c, rd) : (c < NP ? c : (c - NP - rd + NP) % NP));
  }
  __syncthreads();
  // only the pairs this meeting's schedule rotates decide whether it acts
  for (int e = tid; e < JP * JP; e += ROT_THREADS) {
    const int i = e / JP, j = e % JP;
    if (i < j && (full || (i < NP && j >= NP))) {
      const R gii = G[i][i].x, gjj = G[j][j].x, h2 = G[i][j].x * G[i][j].x + G[i][j].y * G[i][j].y;
      if (rot_active<R>(gii, gjj, h2, a.tol, a.neg2)) any_flag = 1;
      if (gii > a.neg2 && gjj > a.neg2 && h2 > a.qtol * gii * gjj) big_lds = 1;
    }
  }
  for (int c = tid; c < JP; c += ROT_THREADS) dd[0][c] = G[c][c].x;
  for (int q = tid; q < NP; q += ROT_THREADS) od[0][q] = G[tb_i[0][q]][tb_j[0][q]];
  __syncthreads();
  if (chunk == 0 && tid == 0 && big_lds) *a.big_cos = 1;
  if (!any_flag) return;
  const R tol_in = R(0.5) * a.tol, neg2 = a.neg2;
  const int rounds = a.max_inner * n_in;
  const bool g_waves = w < 4;          // wave-uniform role
  const int t = tid & 255;
  int buf = 0, round = 0;
  for (int it = 0; it < rounds; ++it) {
    const int nround = round + 1 == n_in ? 0 : round + 1;
    // the round's rotations, once each
    if (tid < NP) {
      const int i = tb_i[round][tid], j = tb_j[round][tid];
      rp[tid] = rot_a(jac_rot(dd[buf][i], dd[buf][j], od[buf][tid], tol_in, neg2));
    }
    __syncthreads();
    const int pb = t % NP;
    const int ib = tb_i[round][pb], jb = tb_j[round][pb];
    const RotA<R> rb = rp[pb];
    if (g_waves) {
#pragma unroll
      for (int k = 0; k < JOBS; ++k) {
        const int pa = (t + 256 * k) / NP;
        const int ia = tb_i[round][pa], ja = tb_j[round][pa];
        const RotA<R> ra = rp[pa];
        C g00 = G[ia][ib], g01 = G[ia][jb], g10 = G[ja][ib], g11 = G[ja][jb];
        rot_right(rb, g00, g01);
        rot_right(rb, g10, g11);
        rot_left(ra, g00, g10);
        rot_left(ra, g01, g11);
        G[ia][ib] = g00;
        G[ia][jb] = g01;
        G[ja][ib] = g10;
        G[ja][jb] = g11;
        // hand on the diagonal and the next round's pair entries
        if (pa == pb) {
          dd[buf ^ 1][ia] = g00.x;
          dd[buf ^ 1][ja] = g11.x;
        }
        const int qa = tb_q[nround][ia], qa2 = tb_q[nround][ja];
        const int qb = tb_q[nround][ib], qb2 = tb_q[nround][jb];
        if (ia < ib && qa == qb) od[buf ^ 1][qa] = g00;
        if (ia < jb && qa == qb2) od[buf ^ 1][qa] = g01;
        if (ja < ib && qa2 == qb) od[buf ^ 1][qa2] = g10;
        if (ja < jb && qa2 == qb2) od[buf ^ 1][qa2] = g11;
      }
    } else {
#pragma unroll
      for (int k = 0; k < JOBS; ++k) {
        const int pa = (t + 256 * k) / NP;
        const int ia = tb_i[round][pa], ja = tb_j[round][pa];
        C v0 = V[ia][ib], v1 = V[ia][jb], v2 = V[ja][ib], v3 = V[ja][jb];
        rot_right(rb, v0, v1);
        rot_right(rb, v2, v3);
        V[ia][ib] = v0;
        V[ia][jb] = v1;
        V[ja][ib] = v2;
        V[ja][jb] = v3;
      }
    }
    buf ^= 1;
    round = nround;
    __syncthreads();
  }
  rotate_rows_by<JP>(a, V, bi, bj, chunk);
}

// The fp32 rotate pass of the cross rounds (all but a sweep's first): the same
// operations on the same values as k_jac_rotate, in the same order, so the
// same bits, without its index tables and with one barrier a round.
// Column q of block bi stays in pair q, and column q of block bj is in pair
// q - r in round r.  Thread (a, b) of waves 0-3 holds the 2 x 2 block of pairs
// a and b and computes pair b's rotation itself (pair a's by a shuffle): of
// its entries (i, i) stays, (i, j) moves one lane down within its 16 lanes,
// and only (j, i), (j, j) and the next rotations' inputs go through LDS.
// Thread (row, b) of waves 4-7 holds V's entries of two rows, which need no LDS
// at all, one round behind.
// Bound: the chain of rounds (0.45 us each) and the launch's loads and stores
// around it (10 us).  1024 x 1024: 21.5 -> 17.8 us a launch.  Tried and no
// faster: the chunk's rows loaded ahead of the solve.
__device__ inline float2 lane_down(float2 v) {   // lane l + 1 of the 16-lane row
  const int x = __builtin_amdgcn_update_dpp(0, __float_as_int(v.x), 0x12f, 0xf, 0xf, false);
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(v.y), 0x12f, 0xf, 0xf, false);
  return make_float2(__int_as_float(x), __int_as_float(y));
}
__global__ __launch_bounds__(ROT_THREADS) void k_jac_rotate_cross(JacArgs<float> a) {
  constexpr int JP = 32, NP = 16;
  __shared__ float2 G[JP][JP + 1];   // the Gram, later V
  __shared__ float2 mji[2][NP][NP], mjj[2][NP][NP];
  __shared__ float dii[2][NP], djj[2][NP];
  __shared__ float2 dij[2][NP];
  __shared__ RotA<float> rp[2][NP];
  __shared__ int any_flag, big_lds;
  const int p = blockIdx.x, chunk = blockIdx.y;
  const int bi = rr_block(p, a.round, a.nbp), bj = rr_block(a.nbp - 1 - p, a.round, a.nbp);
  if (pair_skipped(a, bi, bj)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const float2* part = a.part + (int64_t)p * a.n_gchunks * JP * JP;
  for (int e = tid; e < JP * JP; e += ROT_THREADS) {
    float2 s(0, 0);
    for (int c0 = 0; c0 < a.n_gchunks; c0 += 8) {
      float2 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        t[u] = c0 + u < a.n_gchunks ? part[(int64_t)(c0 + u) * JP * JP + e] : float2(0, 0);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s.x += t[u].x;
        s.y += t[u].y;
      }
    }
    G[e / JP][e % JP] = s;
  }
  if (tid == 0) {
    any_flag = 0;
    big_lds = 0;
  }
  __syncthreads();
  for (int e = tid; e < JP * JP; e += ROT_THREADS) {
    const int i = e / JP, j = e % JP;
    if (i < NP && j >= NP) {
      const float gii = G[i][i].x, gjj = G[j][j].x, h2 = G[i][j].x * G[i][j].x + G[i][j].y * G[i][j].y;
      if (rot_active<float>(gii, gjj, h2, a.tol, a.neg2)) any_flag = 1;
      if (gii > a.neg2 && gjj > a.neg2 && h2 > a.qtol * gii * gjj) big_lds = 1;
    }
  }
  if (tid < NP) {
    dii[0][tid] = G[tid][tid].x;
    djj[0][tid] = G[NP + tid][NP + tid].x;
    dij[0][tid] = G[tid][NP + tid];
  }
  const bool g_waves = tid < 256;
  const int t = tid & 255, pa = t >> 4, pb = t & 15, lane_a = (lane & 48) + pa;
  const int up_a = (pa - 1) & 15, up_b = (pb - 1) & 15;
  // waves 0-3: entries (i, i), (i, j), (j, i), (j, j) of the block; waves 4-7:
  // V's columns i and j of pair b in rows pa and 16 + pa
  float2 x00, x01, x10, x11;
  if (g_waves) {
    x00 = G[pa][pb];
    x01 = G[pa][NP + pb];
    x10 = G[NP + pa][pb];
    x11 = G[NP + pa][NP + pb];
  } else {
    x00 = x11 = make_float2(pa == pb ? 1.0f : 0.0f, 0.0f);
    x01 = x10 = make_float2(0.0f, 0.0f);
  }
  __syncthreads();
  if (chunk == 0 && tid == 0 && big_lds) *a.big_cos = 1;
  if (!any_flag) return;
  const float tol_in = 0.5f * a.tol, neg2 = a.neg2;
  const int rounds = a.max_inner * NP;
  for (int it = 0; it < rounds; ++it) {
    const int buf = it & 1;
    if (g_waves) {
      if (it > 0) {
        x10 = mji[buf][pa][pb];
        x11 = mjj[buf][pa][pb];
      }
      const RotA<float> rb = rot_a(jac_rot(dii[buf][pb], djj[buf][pb], dij[buf][pb], tol_in, neg2));
      RotA<float> ra;
      ra.c = __shfl(rb.c, lane_a);
      ra.ax = __shfl(rb.ax, lane_a);
      ra.ay = __shfl(rb.ay, lane_a);
      if (pa == 0) rp[buf][pb] = rb;
      rot_right(rb, x00, x01);
      rot_right(rb, x10, x11);
      rot_left(ra, x00, x10);
      rot_left(ra, x01, x11);
      mji[buf ^ 1][up_a][pb] = x10;
      mjj[buf ^ 1][up_a][up_b] = x11;
      if (pa == pb) {
        dii[buf ^ 1][pa] = x00.x;
        djj[buf ^ 1][up_a] = x11.x;
      }
      if (up_b == pa) dij[buf ^ 1][pa] = x01;
      x01 = lane_down(x01);
    } else if (it > 0) {
      const RotA<float> rb = rp[buf ^ 1][pb];
      rot_right(rb, x00, x01);
      rot_right(rb, x10, x11);
      x01 = lane_down(x01);
      x11 = lane_down(x11);
    }
    __syncthreads();
  }
  if (!g_waves) {
    const RotA<float> rb = rp[(rounds - 1) & 1][pb];
    rot_right(rb, x00, x01);
    rot_right(rb, x10, x11);
    x01 = lane_down(x01);
    x11 = lane_down(x11);
    G[pa][pb] = x00;
    G[pa][NP + pb] = x01;
    G[NP + pa][pb] = x10;
    G[NP + pa][NP + pb] = x11;
  }
  __syncthreads();
  rotate_rows_by<JP>(a, G, bi, bj, chunk);
}

// Rotate pass with rows in registers (see jacobi_dev.h): waves 0-3 sum the
// partial Grams, solve and publish, the others hold ROWS rows of Y_p.
//
// A sweep's first round takes the pair's whole Gram from the Gram pass.  The
// cross rounds take only the product of the two blocks from it: the blocks'
// own Grams are what the solve of each block's previous meeting left (two
// buffers by the round's parity, since a pair's first workgroup writes the new
// ones while others may still read; every block meets once a round, and the
// last round of a sweep, of which there is an odd number, writes the buffer
// that a skipped pair of the next first round leaves in place).  They drift
// by rounding only and are taken afresh every sweep.  At 2048 x 2048 the Gram
// pass of a cross round takes 13.5 instead of 22.8 us and the rotate pass, with
// a quarter of the partials to read, 28 instead of 32.
template <int ROWS, class S>
__global__ __launch_bounds__(JSOLVE + ROWS) void k_jac_rotate_rows(JacArgs<double> a) {
  __shared__ SolveLds sm;
  constexpr bool kFull = S::rounds == SchedFull::rounds;
  const int p = blockIdx.x, chunk = blockIdx.y;
  const int bi = rr_block(p, a.round, a.nbp), bj = rr_block(a.nbp - 1 - p, a.round, a.nbp);
  const int tid = threadIdx.x;
  const bool skipped = pair_skipped(a, bi, bj);
  const double2* bg_in = a.bg + (int64_t)(a.round & 1) * a.nbp * 256;
  double2* bg_out = a.bg + (int64_t)((a.round & 1) ^ 1) * a.nbp * 256;
  if (skipped) {
    if (!kFull && chunk == 0 && tid < 256) {
      bg_out[bi * 256 + tid] = bg_in[bi * 256 + tid];
      bg_out[bj * 256 + tid] = bg_in[bj * 256 + tid];
    }
    return;
  }
  if (tid >= JSOLVE) {
    const int lane = tid & 63, row = chunk * ROWS + tid - JSOLVE;
    const bool live = row < a.len;
    const int lrow = min(row, a.len - 1);   // unconditional loads: predicated ones would wait one by one
    double2 y[32];
#pragma unroll
    for (int c = 0; c < 32; ++c)
      y[c] = a.x[(int64_t)((c < 16 ? bi : bj) * 16 + (c & 15)) * a.ldx + lrow];
    __syncthreads();                       // Gram summed
    __syncthreads();                       // its pairs checked
    if (!sm.any_flag) return;
    row_sweeps<S>(y, sm, lane, a.max_inner);
    if (live) {
#pragma unroll
      for (int c = 0; c < 32; ++c) {
        double2* col = a.x + (int64_t)((c < 16 ? bi : bj) * 16 + (c & 15)) * a.ldx;
        const double d = column_scale(sm, c);
        col[row] = make_double2(y[c].x * d, y[c].y * d);
      }
    }
    return;
  }
  // partial Grams summed in chunk order, loads issued eight at a time
  constexpr int E = kFull ? 1024 : 256;
  const double2* part = a.part + (int64_t)p * a.n_gchunks * E;
  auto sum_part = [&](int e) {
    double2 s = make_double2(0.0, 0.0);
    for (int c0 = 0; c0 < a.n_gchunks; c0 += 8) {
      double2 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        t[u] = c0 + u < a.n_gchunks ? part[(int64_t)(c0 + u) * E + e] : make_double2(0.0, 0.0);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        s.x += t[u].x;
        s.y += t[u].y;
      }
    }
    return s;
  };
  if constexpr (kFull) {
#pragma unroll
    for (int v = 0; v < 4; ++v) sm.G[tid + JSOLVE * v] = sum_part(tid + JSOLVE * v);
  } else {
    const int m = tid >> 4, n = tid & 15;
    const double2 gi = bg_in[bi * 256 + tid], gj = bg_in[bj * 256 + tid];
    const double2 s = sum_part(tid);
    sm.G[m * 32 + n] = gi;
    sm.G[(16 + m) * 32 + 16 + n] = gj;
    sm.G[m * 32 + 16 + n] = s;
    sm.G[(16 + n) * 32 + m] = make_double2(s.x, -s.y);
  }
  fill_schedule<S>(sm, tid, JSOLVE);
  const Moves<S> moves = block_moves<S>(tid);
  if (tid < 32) {
    sm.scale[tid] = 1.0;
    sm.scale_err[tid] = 0.0;
  }
  if (tid == 0) {
    sm.any_flag = 0;
    sm.big = 0;
  }
  __syncthreads();
  load_blocks<S>(sm, tid);
  // only the pairs this meeting's schedule rotates decide whether it acts
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int e = tid + JSOLVE * v, i = e >> 5, j = e & 31;
    if (i < j && (kFull || (i < 16 && j >= 16))) {
      const double gii = sm.G[33 * i].x, gjj = sm.G[33 * j].x;
      const double2 g = sm.G[e];
      const double h2 = g.x * g.x + g.y * g.y;
      if (rot_active<double>(gii, gjj, h2, a.tol, a.neg2)) sm.any_flag = 1;
      if (gii > a.neg2 && gjj > a.neg2 && h2 > a.qtol * gii * gjj) sm.big = 1;
    }
  }
  __syncthreads();
  if (chunk == 0 && tid == 0 && sm.big) *a.big_cos = 1;
  if (!sm.any_flag) {
    if (chunk == 0) {
      const int m = tid >> 4, n = tid & 15;
      bg_out[bi * 256 + tid] = sm.G[m * 32 + n];
      bg_out[bj * 256 + tid] = sm.G[(16 + m) * 32 + 16 + n];
    }
    return;
  }
  solve_sweeps<S>(sm, moves, tid, 0.5 * a.tol, a.neg2, a.max_inner);
  if (chunk == 0) {
    // the blocks' Grams: the solve's copy is back in the order of round 0
    if (tid < Blocks<S>::n) {
      const int qb = tid & 15, qa = (qb + tid / 16) & 15, buf = (a.max_inner * S::rounds) & 1;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int r = t >= 2 ? S::j(qa, 0) : S::i(qa, 0), c = t & 1 ? S::j(qb, 0) : S::i(qb, 0);
        if ((r ^ c) & 16 || (t == 2 && tid < 16)) continue;   // between the blocks, or not kept
        const double2 g = sm.B[buf][t][tid];
        double2* out = bg_out + (r < 16 ? bi : bj) * 256;
        out[(r & 15) * 16 + (c & 15)] = g;
        if (r != c) out[(c & 15) * 16 + (r & 15)] = make_double2(g.x, -g.y);
      }
    }
    if (tid == 0) {
      a.rot_cur[bi] = 1;
      a.rot_cur[bj] = 1;
      atomicAdd(a.rot_count, 1);
    }
  }
}

// rot_prev <- rot_cur (or all ones before the first sweep), rot_cur <- 0,
// rot_count <- 0, big_cos <- 0.
__global__ void k_jac_roll(int* rot_prev, int* rot_cur, int* rot_count, int* big_cos, int nbp, int first) {
  for (int i = threadIdx.x; i < nbp; i += blockDim.x) {
    rot_prev[i] = first ? 1 : rot_cur[i];
    rot_cur[i] = 0;
  }
  if (threadIdx.x == 0) {
    *rot_count = 0;
    *big_cos = 0;
  }
}

// ------------------------------------------------------------- driver
bool jacobi_debug() {
  static const bool v = [] {
    const char* e = std::getenv("RCS_DEBUG_JACOBI");
    return e && e[0] == '1';
  }();
  return v;
}

// Tuning table: buckets (cnt_max ascending) -> block width, inner sweeps.
namespace {
struct TuneEntry {
  int cnt_max, jb, inner;
};
std::vector<TuneEntry> g_tune;
std::mutex g_tune_mu;
}  // namespace

void tuning_set(int cnt_max, int jb, int inner) {
  RCS_REQUIRE(jb == 16 || jb == 32, "block width must be 16 or 32");
  RCS_REQUIRE(inner >= 1 && inner <= 8, "inner sweeps must be in [1, 8]");
  std::lock_guard<std::mutex> lk(g_tune_mu);
  for (auto& e : g_tune)
    if (e.cnt_max == cnt_max) {
      e.jb = jb;
      e.inner = inner;
      return;
    }
  g_tune.push_back({cnt_max, jb, inner});
  std::sort(g_tune.begin(), g_tune.end(), [](const TuneEntry& a, const TuneEntry& b) { return a.cnt_max < b.cnt_max; });
}

void tuning_clear() {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune.clear();
}

static void tuned(int cnt, int* jb, int* inner) {
  *jb = 16;
  *inner = 1;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (const auto& e : g_tune)
      if (cnt <= e.cnt_max) {
        *jb = e.jb;
        *inner = e.inner;
        break;
      }
  }
  const char* b = std::getenv("RCS_JACOBI_BLOCK");
  if (b && (std::atoi(b) == 16 || std::atoi(b) == 32)) *jb = std::atoi(b);
  const char* i = std::getenv("RCS_JACOBI_INNER");
  if (i && std::atoi(i) >= 1 && std::atoi(i) <= 8) *inner = std::atoi(i);
}

// Waves of a Gram workgroup.
static int gram_waves(const JacobiPlan& pl, bool f32) { return pl.jb == 16 && !f32 && pl.len > 768 ? 8 : 4; }

JacobiPlan jacobi_plan(int len, int cnt, int jb, bool f32) {
  JacobiPlan pl;
  int tjb, tin;
  tuned(cnt, &tjb, &tin);
  if (jb <= 0) jb = tjb;
  pl.inner = tin;
  RCS_REQUIRE(jb == 16 || jb == 32, "Jacobi block must be 16 or 32 columns");
  pl.jb = jb;
  pl.len = len;
  pl.cnt = cnt;
  pl.ldx = (int)round_up(std::max(len, 1), 64);
  int nb = ceil_div(std::max(cnt, 1), jb);
  pl.nbp = std::max(2, nb + (nb & 1));
  pl.cnt_pad = pl.nbp * jb;
  pl.n_pairs = pl.nbp / 2;
  static const int wgs = [] {
    const char* e = std::getenv("RCS_JACOBI_WGS");
    const int v = e ? std::atoi(e) : 0;
    return v >= 64 && v <= 4096 ? v : 256;
  }();
  const int target_chunks = std::max(1, wgs / pl.n_pairs);
  const int max_chunks = ceil_div(len, 64);
  pl.n_chunks = std::max(1, std::min(target_chunks, max_chunks));
  pl.rows_per_chunk = (int)round_up(ceil_div(len, pl.n_chunks), TR);
  pl.n_chunks = ceil_div(len, pl.rows_per_chunk);
  // Gram chunks: two workgroups per compute unit hide each other's loads
  if (gram_waves(pl, f32) == 8)
    pl.n_gchunks = std::max(1, std::min(512 / pl.n_pairs, ceil_div(len, 128)));
  else
    pl.n_gchunks = std::max(1, std::min(2 * pl.n_chunks, max_chunks));
  pl.rows_per_gchunk = (int)round_up(ceil_div(len, pl.n_gchunks), TR);
  pl.n_gchunks = ceil_div(len, pl.rows_per_gchunk);
  return pl;
}

size_t jacobi_work_bytes(const JacobiPlan& pl) {
  const int JP = 2 * pl.jb;
  return ((size_t)pl.n_pairs * pl.n_gchunks * JP * JP + 2 * (size_t)pl.nbp * 256) * sizeof(double2) +
         2 * (size_t)pl.nbp * sizeof(int) + 256;
}

// Row-resident rotate pass: the fewest rows per workgroup (64 to 512) that
// leave at most one workgroup per compute unit.
static int rows_per_wg(const JacobiPlan& pl) {
  for (int rows = 64; rows < 512; rows *= 2)
    if ((int64_t)pl.n_pairs * ceil_div(pl.len, rows) <= 256) return rows;
  return 512;
}
template <int ROWS>
static void launch_rotate_rows_n(const JacobiPlan& pl, const JacArgs<double>& a, hipStream_t stream, hipEvent_t start,
                                 hipEvent_t stop) {
  const dim3 grid(pl.n_pairs, ceil_div(pl.len, ROWS)), block(JSOLVE + ROWS);
  if (a.round == 0)
    hipExtLaunchKernelGGL((k_jac_rotate_rows<ROWS, SchedFull>), grid, block, 0, stream, start, stop, 0, a);
  else
    hipExtLaunchKernelGGL((k_jac_rotate_rows<ROWS, SchedCross>), grid, block, 0, stream, start, stop, 0, a);
}
static void launch_rotate_rows(const JacobiPlan& pl, const JacArgs<double>& a, hipStream_t stream, hipEvent_t start,
                               hipEvent_t stop) {
  switch (rows_per_wg(pl)) {
    case 64: launch_rotate_rows_n<64>(pl, a, stream, start, stop); break;
    case 128: launch_rotate_rows_n<128>(pl, a, stream, start, stop); break;
    case 256: launch_rotate_rows_n<256>(pl, a, stream, start, stop); break;
    default: launch_rotate_rows_n<512>(pl, a, stream, start, stop);
  }
}

template <typename R>
static void launch_sweep(const JacobiPlan& pl, JacArgs<R> a, hipStream_t stream, bool first) {
  hipLaunchKernelGGL(k_jac_roll, dim3(1), dim3(256), 0, stream, a.rot_prev, a.rot_cur, a.rot_count, a.big_cos, pl.nbp,
                     first ? 1 : 0);
  HIP_LAUNCH_OK();
  for (int r = 0; r < pl.nbp - 1; ++r) {
    a.round = r;
    // nominal algorithmic work of a round with every pair active: Gram and
    // update are each n_pairs complex GEMMs of len x JP x JP
    const double JPd = 2.0 * pl.jb;
    const double fl = 8.0 * pl.len * JPd * JPd * pl.n_pairs;
    const double by = 16.0 * (double)pl.len * JPd * pl.n_pairs;
    {
      Probe pr(kKcJacGram, stream, fl, by);
      const int waves = gram_waves(pl, std::is_same<R, float>::value);
      const dim3 grid(pl.n_pairs, pl.n_gchunks), block(64 * waves);
      auto launch = [&](auto kernel) { hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, pr.start(), pr.stop(), 0, a); };
      bool cross = false;   // the row-resident pass takes only the cross products after a sweep's first round
      if constexpr (std::is_same<R, double>::value) {
        cross = pl.jb == 16 && r > 0;
        if (cross && waves == 8)
          launch(k_jac_gram<32, 8, R, true>);
        else if (cross)
          launch(k_jac_gram<32, 4, R, true>);
      }
      if (!cross) {
        if (pl.jb != 16)
          launch(k_jac_gram<64, 4, R>);
        else if (waves == 8)
          launch(k_jac_gram<32, 8, R>);
        else
          launch(k_jac_gram<32, 4, R>);
      }
    }
    HIP_LAUNCH_OK();
    {
      Probe pr(kKcJacRotate, stream, fl, 2.0 * by);
      if (pl.jb != 16)
        hipExtLaunchKernelGGL((k_jac_rotate<64, R>), dim3(pl.n_pairs, pl.n_chunks), dim3(ROT_THREADS), 0, stream,
                              pr.start(), pr.stop(), 0, a);
      else if constexpr (std::is_same<R, double>::value)
        launch_rotate_rows(pl, a, stream, pr.start(), pr.stop());
      else if (r == 0)
        hipExtLaunchKernelGGL((k_jac_rotate<32, R>), dim3(pl.n_pairs, pl.n_chunks), dim3(ROT_THREADS), 0, stream,
                              pr.start(), pr.stop(), 0, a);
      else
        hipExtLaunchKernelGGL(k_jac_rotate_cross, dim3(pl.n_pairs, pl.n_chunks), dim3(ROT_THREADS), 0, stream,
                              pr.start(), pr.stop(), 0, a);
    }
    HIP_LAUNCH_OK();
  }
}

// Stop after a sweep whose largest entering squared cosine c2 satisfies
// f c2 <= tol, f = 100 (RCS_JACOBI_QSTOP overrides; 0 turns it off): the
// Jacobi iteration converges quadratically at the end, so the next sweep
// would start below ~c2 and rotate nothing; it is not run.  On the
// 53-qubit chi 1024 build this skips 1,016 of 1,278 such verification
// sweeps, and in none of the skipped cases did the sweep rotate anything
// when run.
static double jacobi_qstop() {
  static const double v = [] {
    const char* e = std::getenv("RCS_JACOBI_QSTOP");
    const double f = e ? std::atof(e) : 100.0;
    return f > 0.0 ? f : 0.0;
  }();
  return v;
}

static JacobiTol jacobi_tol_u(double u, int len, double tol) {
  JacobiTol t;
  t.tol = tol > 0.0 ? tol : 16.0 * u * std::sqrt((double)std::max(len, 16));
  // columns shorter than delta ||X||_F (delta = 8 u sqrt(len)) are numerically
  // zero: below the absolute accuracy of any SVD in this precision, and they
  // must not be required to be mutually orthogonal (a wide matrix has more
  // columns than its rank)
  const double delta = 8.0 * u * std::sqrt((double)len);
  t.delta2 = delta * delta;
  t.qtol = jacobi_qstop() > 0.0 ? t.tol / jacobi_qstop() : 0.0;
  return t;
}
JacobiTol jacobi_tol(int len, double tol) { return jacobi_tol_u(JT<double>::u, len, tol); }

static bool use_graphs() {
  static const bool v = [] {
    const char* e = std::getenv("RCS_JACOBI_GRAPH");
    return e && e[0] == '1';
  }();
  return v;
}

// One sweep (not the first) as an executable graph.  It belongs to one run: the
// launches it replays carry that matrix's addresses and thresholds.
struct SweepGraph {
  hipGraphExec_t exec = nullptr;
  SweepGraph() = default;
  SweepGraph(const SweepGraph&) = delete;
  SweepGraph& operator=(const SweepGraph&) = delete;
  ~SweepGraph() {
    if (exec) (void)hipGraphExecDestroy(exec);
  }
  void launch(const JacobiPlan& pl, const JacArgs<double>& a, hipStream_t stream) {
    if (!exec) capture(pl, a);
    HIP_OK(hipGraphLaunch(exec, stream));
  }

 private:
  void capture(const JacobiPlan& pl, const JacArgs<double>& a) {
    hipStream_t cs;
    HIP_OK(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      try {
        launch_sweep(pl, a, cs, false);
      } catch (...) {
        (void)hipStreamEndCapture(cs, &graph);
        if (graph) (void)hipGraphDestroy(graph);
        (void)hipStreamDestroy(cs);
        throw;
      }
      e = hipStreamEndCapture(cs, &graph);
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(cs);
    HIP_OK(e);
  }
};

// x *= 2^e, exactly (up to underflow).
__global__ void k_jac_scale(double2* x, int64_t n, int e) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] = make_double2(ldexp(x[i].x, e), ldexp(x[i].y, e));
}
static void jac_scale(const JacobiPlan& pl, double2* x, int e, hipStream_t s) {
  const int64_t n = (int64_t)pl.ldx * pl.cnt_pad;
  hipLaunchKernelGGL(k_jac_scale, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65535)), dim3(256), 0, s, x, n, e);
  HIP_LAUNCH_OK();
}
// The exponent by which the fp64 iteration scales its columns: 0 where
// ||x||_F^2 is within 2^(+-300).  The rotations form products of two Gram
// entries next to an addend of 1e-300 (jac_rot_t): beyond 2^512 they overflow,
// and the smallest ones that matter (cosines at the tolerance between columns
// at the zero level, about 1e-88 fro2^2) stay clear of the addend down to
// 2^-320.  A power of two leaves every rounding of the iteration alike.
static int jac_scale_exponent(double fro2) {
  if (!(fro2 > 0.0) || !std::isfinite(fro2) || (fro2 >= 0x1p-300 && fro2 <= 0x1p300)) return 0;
  return -(int)std::floor(0.5 * std::ilogb(fro2));
}

template <typename R>
static int jacobi_run_t(const JacobiPlan& pl, typename JT<R>::C* x, void* work, int* rot_count_dev,
                        int* rot_count_host, double fro2, hipStream_t stream, int max_sweeps, double tol) {
  using C = typename JT<R>::C;
  JacArgs<R> a;
  a.x = x;
  a.ldx = pl.ldx;
  a.len = pl.len;
  a.nbp = pl.nbp;
  a.rows_per_chunk = pl.rows_per_chunk;
  a.n_chunks = pl.n_chunks;
  a.rows_per_gchunk = pl.rows_per_gchunk;
  a.n_gchunks = pl.n_gchunks;
  a.round = 0;
  char* w = reinterpret_cast<char*>(work);
  a.part = reinterpret_cast<C*>(w);
  w += (size_t)pl.n_pairs * pl.n_gchunks * (2 * pl.jb) * (2 * pl.jb) * sizeof(C);
  a.bg = reinterpret_cast<C*>(w);
  w += 2 * (size_t)pl.nbp * 256 * sizeof(C);
  a.rot_prev = reinterpret_cast<int*>(w);
  a.rot_cur = a.rot_prev + pl.nbp;
  a.rot_count = rot_count_dev;
  a.big_cos = rot_count_dev + 1;
  const JacobiTol t = jacobi_tol_u(JT<R>::u, pl.len, tol);
  a.tol = (R)t.tol;
  a.neg2 = (R)(t.delta2 * std::max(fro2, 1e-300));
  a.qtol = (R)(jacobi_qstop() > 0.0 ? (double)a.tol / jacobi_qstop() : 0.0);
  a.max_inner = pl.inner;
  [[maybe_unused]] const bool graphs = use_graphs() && pl.nbp > 4;
  [[maybe_unused]] SweepGraph graph;
  for (int sweep = 1; sweep <= max_sweeps; ++sweep) {
    if constexpr (std::is_same<R, double>::value) {
      if (graphs && sweep > 1)
        graph.launch(pl, a, stream);
      else
        launch_sweep(pl, a, stream, sweep == 1);
    } else {
      launch_sweep(pl, a, stream, sweep == 1);
    }
    HIP_OK(hipMemcpyAsync(rot_count_host, rot_count_dev, 2 * sizeof(int), hipMemcpyDeviceToHost, stream));
    HIP_OK(hipStreamSynchronize(stream));
    const bool big = rot_count_host[1] != 0;
    if (jacobi_debug())
      std::fprintf(stderr, "jacobi %dx%d sweep %d: %d pair rotations%s\n", pl.len, pl.cnt, sweep, *rot_count_host,
                   big ? "" : ", all entering cosines below the quadratic-stop level");
    if (*rot_count_host == 0) return sweep;
    // quadratic convergence: after a sweep whose meetings all entered with
    // squared cosines below tol / f, the next one starts below ~tol^2 / f^2
    if (jacobi_qstop() > 0.0 && !big) return sweep;
  }
  fail(RCS_ERR_NUMERIC, "one-sided Jacobi SVD did not converge");
}

int jacobi_run(const JacobiPlan& pl, double2* x, void* work, int* rot_count_dev, int* rot_count_host, double fro2,
               hipStream_t stream, int max_sweeps, double tol) {
  const int e = jac_scale_exponent(fro2);
  if (e) jac_scale(pl, x, e, stream);
  const int sweeps = jacobi_run_t<double>(pl, x, work, rot_count_dev, rot_count_host, std::ldexp(fro2, 2 * e), stream,
                                          max_sweeps, tol);
  if (e) jac_scale(pl, x, -e, stream);
  return sweeps;
}

int jacobi_run_f32(const JacobiPlan& pl, float2* x, void* work, int* rot_count_dev, int* rot_count_host, double fro2,
                   hipStream_t stream, int max_sweeps, double tol) {
  return jacobi_run_t<float>(pl, x, work, rot_count_dev, rot_count_host, fro2, stream, max_sweeps, tol);
}

}  // namespace rcs

extern "C" {

rcs_status rcs_tuning_set(int32_t cnt_max, int32_t block, int32_t inner_sweeps) {
  try {
    rcs::tuning_set(cnt_max, block, inner_sweeps);
  } catch (const rcs::Error& e) {
    rcs::set_last_error(e.what());
    return e.status;
  } catch (const std::bad_alloc&) {
    rcs::set_last_error("host allocation failed");
    return RCS_ERR_OUT_OF_MEMORY;
  } catch (const std::exception& e) {
    rcs::set_last_error(e.what());
    return RCS_ERR_DEVICE;
  }
  return RCS_OK;
}

void rcs_tuning_clear(void) { rcs::tuning_clear(); }

}  // extern "C"
