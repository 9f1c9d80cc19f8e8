// Split of a small two-site matrix (up to 128 x 32) in one launch: Jacobi SVD,
// rank rule, normalisation, Newton-Schulz and projection by one workgroup.
//
// Near the ends of a chain the matrices are small, and the general split's
// launches (two per round, about fifteen around them) and one wait of the
// host per sweep cost far more than its arithmetic.  Here rows 0-127 sit in
// the registers of waves 4 and 5 throughout (one row per lane), the Gram is
// taken from an LDS copy of them on the matrix cores (3.4 us at 128 x 32),
// and waves 0-3 solve it and publish; jacobi_dev.h has the scheme.  One sweep
// is a round robin over all 8, 16 or 32 columns, so the Gram is fresh once a
// sweep, as in the general path with one column block.
// Bound: the chain of rounds (0.48 us each, 31 a sweep at 32 columns).
// Measured, kernel time at 8 / 16 / 32 columns in an exact 12-qubit build:
// 19 / 58 / 180 us, where the general split's 35 or so launches and its wait
// per sweep took about 380 us; the whole build 48.0 -> 23.7 ms.  The factors
// go straight into the site tensors and the rank into pinned host memory,
// which saves two launches an update and three a move (17.4 -> 16.4 ms).
//
// Range: what one workgroup's registers hold, 128 rows of 32 columns.  That
// covers every split with a neighbouring bond of at most 16; a 64-column
// matrix is two column blocks, i.e. the general path's pairs.
#include "jacobi_dev.h"
#include "prof.h"
#include "split_small.h"

namespace rcs {

constexpr int SS_THREADS = JSOLVE + kSplitSmallRows;
constexpr int SS_LD = kSplitSmallRows + 1;   // odd: 16 columns x 4 rows of an MFMA operand spread over the banks

template <int N>
struct SmallDims {
  static constexpr int cols = N < 16 ? 16 : N;       // whole 16-column tiles
  static constexpr int nb = cols / 16;
  static constexpr int tiles = nb * (nb + 1) / 2;    // of the upper triangle
  static constexpr int kparts = tiles == 3 ? 2 : 4;  // waves per tile
};

template <int N>
struct SmallLds {
  SolveLds sv;
  double2 Y[SmallDims<N>::cols * SS_LD];
  double part[SmallDims<N>::tiles * SmallDims<N>::kparts][8][64];
  double key[32], sorted[32];
  int order[32];
  int bad;
  RankOut rk;
};

// G = Y^H Y over the first len rows (those from len on are zero), by all waves.
template <int N>
__device__ inline void small_gram(SmallLds<N>& sm, int len, int tid) {
  using D = SmallDims<N>;
  using T = JT<double>;
  const int lane = tid & 63, w = tid >> 6;
  if (w < D::tiles * D::kparts) {
    const int u = w % D::tiles, kp = w / D::tiles;
    const int mb = u == 2 ? 1 : 0, nb = u == 0 ? 0 : 1;
    double4_t gr{0, 0, 0, 0}, gi{0, 0, 0, 0};
    const int c = lane & 15, steps = (len + 3) / 4;
    const double2* ym = sm.Y + (mb * 16 + c) * SS_LD + (lane >> 4);
    const double2* yn = sm.Y + (nb * 16 + c) * SS_LD + (lane >> 4);
    for (int ks = kp; ks < steps; ks += D::kparts) {
      const double2 a = ym[4 * ks], b = yn[4 * ks];
      gr = T::mma(a.x, b.x, gr);
      gi = T::mma(a.x, b.y, gi);
      gr = T::mma(a.y, b.y, gr);
      gi = T::mma(-a.y, b.x, gi);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sm.part[u * D::kparts + kp][r][lane] = gr[r];
      sm.part[u * D::kparts + kp][4 + r][lane] = gi[r];
    }
  }
  __syncthreads();
  double2* G = sm.sv.G;
  for (int e = tid; e < D::tiles * 256; e += SS_THREADS) {
    const int u = e >> 8, r = (e >> 6) & 3, l = e & 63;
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int kp = 0; kp < D::kparts; ++kp) {
      re += sm.part[u * D::kparts + kp][r][l];
      im += sm.part[u * D::kparts + kp][4 + r][l];
    }
    const int m = (u == 2 ? 16 : 0) + T::orow(l, r), n = (u == 0 ? 0 : 16) + (l & 15);
    G[m * 32 + n] = make_double2(re, im);
    if (u == 1) G[n * 32 + m] = make_double2(re, -im);
  }
  __syncthreads();
}

// Y <- Y H, H (cols x cols) in G; a wave's 16-row tiles depend only on
// their own rows, so the product is in place.
template <int N>
__device__ inline void small_apply(SmallLds<N>& sm, int len, int tid) {
  using D = SmallDims<N>;
  using T = JT<double>;
  const int lane = tid & 63, w = tid >> 6, c = lane & 15;
  if (w < 4) {
    const double2* H = sm.sv.G;
    for (int rt = w; rt * 16 < len; rt += 4) {
      double4_t re[D::nb], im[D::nb];
#pragma unroll
      for (int nb = 0; nb < D::nb; ++nb) re[nb] = im[nb] = double4_t{0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < D::cols / 4; ++ks) {
        const int k = 4 * ks + (lane >> 4);
        const double2 a = sm.Y[k * SS_LD + rt * 16 + c];
#pragma unroll
        for (int nb = 0; nb < D::nb; ++nb) {
          const double2 b = H[k * 32 + nb * 16 + c];
          re[nb] = T::mma(a.x, b.x, re[nb]);
          im[nb] = T::mma(a.x, b.y, im[nb]);
          re[nb] = T::mma(-a.y, b.y, re[nb]);
          im[nb] = T::mma(a.y, b.x, im[nb]);
        }
      }
#pragma unroll
      for (int nb = 0; nb < D::nb; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sm.Y[(nb * 16 + c) * SS_LD + rt * 16 + T::orow(lane, r)] = make_double2(re[nb][r], im[nb][r]);
    }
  }
  __syncthreads();
}

// G <- (3 I - G) / 2
template <int N>
__device__ inline void small_ns(SmallLds<N>& sm, int tid) {
  double2* H = sm.sv.G;
  for (int e = tid; e < 32 * SmallDims<N>::cols; e += SS_THREADS) {
    const int i = e >> 5, j = e & 31;
    if (j < SmallDims<N>::cols) H[e] = make_double2((i == j ? 1.5 : 0.0) - 0.5 * H[e].x, -0.5 * H[e].y);
  }
  __syncthreads();
}

// P (k x cnt) = scale Y^H X, X from memory (load(row, column)); one wave per
// 16 x 16 tile, elements passed to store(m, c, v).
template <int N, class Load, class Store>
__device__ inline void small_project(const SmallLds<N>& sm, int len, int cnt, int k, double scale, int tid,
                                     const Load& load, const Store& store) {
  using D = SmallDims<N>;
  using T = JT<double>;
  const int lane = tid & 63, w = tid >> 6;
  if (w >= D::nb * D::nb) return;
  const int m0 = (w / D::nb) * 16, n0 = (w % D::nb) * 16;
  if (m0 >= k || n0 >= cnt) return;
  const int c = n0 + (lane & 15), rsub = lane >> 4;
  const int lc = min(c, cnt - 1);   // columns from cnt on are not stored
  const double2* y = sm.Y + (m0 + (lane & 15)) * SS_LD;
  double4_t re{0, 0, 0, 0}, im{0, 0, 0, 0};
  for (int r0 = 0; r0 < len; r0 += 32) {
    double2 b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) b[q] = load(min(r0 + 4 * q + rsub, len - 1), lc);   // Y is zero from len on
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double2 v = y[r0 + 4 * q + rsub];
      re = T::mma(v.x, b[q].x, re);
      im = T::mma(v.x, b[q].y, im);
      re = T::mma(v.y, b[q].y, re);
      im = T::mma(-v.y, b[q].x, im);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = m0 + T::orow(lane, r);
    if (m < k && c < cnt) store(m, c, make_double2(re[r] * scale, im[r] * scale));
  }
}

// order[] <- indices of key[0..n) descending, ties by index (one thread per
// key; NaN keys leave some of order[] at its previous content).
__device__ inline void rank_keys(const double* key, int n, int* order, int tid) {
  if (tid < n) {
    const double v = key[tid];
    int rank = 0;
    for (int j = 0; j < n; ++j) rank += key[j] > v || (key[j] == v && j < tid);
    order[rank] = tid;
  }
}

// The rank rule of k_sort_rank, with its order of sums, on keys in registers.
template <int N>
__device__ inline RankOut rank_rule(const double* sorted, int cnt, int cap, double eps) {
  double s2[N];
#pragma unroll
  for (int i = 0; i < N; ++i) s2[i] = i < cnt ? sorted[i] * sorted[i] : 0.0;
  double w = 0.0;
#pragma unroll
  for (int i = N - 1; i >= 0; --i) w += s2[i];
  const double floor = 1e-24 * w;
  int nnz = 0, k_eps = cnt;
#pragma unroll
  for (int i = 0; i < N; ++i) nnz = i < cnt && s2[i] > floor ? i + 1 : nnz;
  double tail = 0.0, tail_k = 0.0;
  bool open = true;
#pragma unroll
  for (int k = N; k >= 1; --k) {
    open = open && tail <= eps * w;
    if (open && k <= cnt) {
      k_eps = k;
      tail_k = tail;
    }
    tail += s2[k - 1] <= floor ? 0.0 : s2[k - 1];
  }
  RankOut o;
  o.k = min(k_eps, cap);
  double tk = 0.0, kept = 0.0;
#pragma unroll
  for (int i = N - 1; i >= 0; --i) tk += i < o.k || s2[i] <= floor ? 0.0 : s2[i];
#pragma unroll
  for (int i = 0; i < N; ++i) kept += i < o.k ? s2[i] : 0.0;
  if (o.k == k_eps) tk = tail_k;
  o.nnz = nnz;
  o.eps_step = w > 0.0 ? tk / w : 0.0;
  o.w = w;
  o.nrm = sqrt(kept);
  o.bad = !(w > 0.0);
  return o;
}

template <int N>
__global__ __launch_bounds__(SS_THREADS) void k_split_small(SplitSmallArgs a) {
  using S = SchedRR<N>;
  using D = SmallDims<N>;
  __shared__ SmallLds<N> sm;
  const int tid = threadIdx.x, lane = tid & 63, row = tid - JSOLVE;
  const bool row_wave = tid >= JSOLVE;
  const Moves<S> moves = block_moves<S>(tid);
  double2 y[N];
  if (row_wave) {
    const int lrow = min(row, a.len - 1);
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const double2 v = a.x[(int64_t)min(c, a.cnt - 1) * a.ldx + lrow];
      y[c] = c < a.cnt && row < a.len ? v : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int c = 0; c < D::cols; ++c) sm.Y[c * SS_LD + row] = c < N ? y[c < N ? c : 0] : make_double2(0.0, 0.0);
  } else {
    fill_schedule<S>(sm.sv, tid, JSOLVE);
    if (tid < 32) {
      sm.sv.scale[tid] = 1.0;
      sm.sv.scale_err[tid] = 0.0;
      sm.order[tid] = tid;
    }
    if (tid == 0) sm.sv.any_flag = sm.sv.big = sm.bad = 0;
  }
  __syncthreads();
  small_gram(sm, a.len, tid);
  // columns by norm
  double fro2 = 0.0;
#pragma unroll
  for (int c = 0; c < N; ++c) fro2 += sm.sv.G[33 * c].x;
  const double neg2 = a.delta2 * fmax(fro2, 1e-300);
  if (tid < 32) sm.key[tid] = sm.sv.G[33 * tid].x;
  __syncthreads();
  if (a.sort) rank_keys(sm.key, a.cnt, sm.order, tid);
  __syncthreads();
  if (row_wave) {
#pragma unroll
    for (int c = 0; c < N; ++c) y[c] = sm.Y[sm.order[c] * SS_LD + row];
#pragma unroll
    for (int c = 0; c < N; ++c) sm.Y[c * SS_LD + row] = y[c];
  }
  constexpr int GP = (32 * N + SS_THREADS - 1) / SS_THREADS;
  double2 g[GP];
#pragma unroll
  for (int v = 0; v < GP; ++v) {
    const int e = tid + SS_THREADS * v, i = (e >> 5) & (N - 1), j = e & 31;
    g[v] = sm.sv.G[sm.order[i] * 32 + sm.order[j]];
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < GP; ++v)
    if (tid + SS_THREADS * v < 32 * N) sm.sv.G[tid + SS_THREADS * v] = g[v];
  __syncthreads();
  int sweeps = 0;
  for (;;) {
    if (!row_wave) load_blocks<S>(sm.sv, tid);
    for (int e = tid; e < 32 * N; e += SS_THREADS) {
      const int i = e >> 5, j = e & 31;
      if (i < j && j < N) {
        const double gii = sm.sv.G[33 * i].x, gjj = sm.sv.G[33 * j].x;
        const double2 g = sm.sv.G[e];
        const double h2 = g.x * g.x + g.y * g.y;
        if (rot_active<double>(gii, gjj, h2, a.tol, neg2)) sm.sv.any_flag = 1;
        if (gii > neg2 && gjj > neg2 && h2 > a.qtol * gii * gjj) sm.sv.big = 1;
      }
    }
    __syncthreads();
    const bool any = sm.sv.any_flag != 0, big = sm.sv.big != 0;
    ++sweeps;
    if (!any) break;
    if (row_wave) {
      row_sweeps<S>(y, sm.sv, lane, 1);
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const double d = column_scale(sm.sv, c);
        y[c] = make_double2(y[c].x * d, y[c].y * d);
        sm.Y[c * SS_LD + row] = y[c];
      }
    } else {
      solve_sweeps<S>(sm.sv, moves, tid, 0.5 * a.tol, neg2, 1);
    }
    __syncthreads();
    if (tid < 32) {
      sm.sv.scale[tid] = 1.0;
      sm.sv.scale_err[tid] = 0.0;
    }
    if (tid == 0) sm.sv.any_flag = sm.sv.big = 0;
    small_gram(sm, a.len, tid);
    if (a.qtol > 0.0 && !big) break;
    if (sweeps == a.max_sweeps) {
      sweeps = -1;
      break;
    }
  }
  // singular values and rank
  if (tid < 32) {
    const double s = sqrt(sm.sv.G[33 * (tid < N ? tid : 0)].x);
    sm.key[tid] = s;
    sm.order[tid] = tid;
    if (tid < a.cnt && (!(s == s) || s > 1e300)) sm.bad = 1;
  }
  __syncthreads();
  rank_keys(sm.key, a.cnt, sm.order, tid);
  __syncthreads();
  if (tid < a.cnt) {
    const double s = sm.key[sm.order[tid]];
    sm.sorted[tid] = s;
    a.sorted[tid] = s;
  }
  __syncthreads();
  if (tid == 0) {
    RankOut o = rank_rule<N>(sm.sorted, a.cnt, a.cap, a.eps);
    o.bad |= sm.bad;
    o.sweeps = sweeps;
    sm.rk = o;
    *a.out = o;
  }
  __syncthreads();
  const int k = sm.rk.k;
  if (row_wave) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const double2 v = sm.Y[sm.order[j] * SS_LD + row];
      const double inv = j < k ? 1.0 / sm.sorted[j < k ? j : 0] : 0.0;
      y[j] = make_double2(v.x * inv, v.y * inv);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) sm.Y[j * SS_LD + row] = j < k ? y[j] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  for (int it = 0; it < a.ns_steps; ++it) {
    small_gram(sm, a.len, tid);
    small_ns(sm, tid);
    small_apply(sm, a.len, tid);
  }
  const auto load = [&](int r, int c) { return a.x[(int64_t)c * a.ldx + r]; };
  const double scale = a.renorm ? 1.0 / sm.rk.nrm : 1.0;
  if (!a.ai) {
    if (row_wave) {
      if (row < a.len)
        for (int j = 0; j < k; ++j) a.wn[(int64_t)j * a.ldx + row] = sm.Y[j * SS_LD + row];
    } else {
      small_project(sm, a.len, a.cnt, k, scale, tid, load,
                    [&](int m, int c, double2 v) { a.p[(int64_t)m * a.cnt + c] = v; });
    }
    return;
  }
  // row (s, a) of ai's side and column j, row (s, c) of aj's side and j
  auto left = [&](int r, int j, double2 v) { a.ai[(int64_t)r * k + j] = v; };
  auto right = [&](int r, int j, double2 v) {
    const int s = r >= a.dr ? 1 : 0;
    a.aj[((int64_t)s * k + j) * a.dr + r - s * a.dr] = v;
  };
  auto conj = [](double2 v) { return make_double2(v.x, -v.y); };
  if (row_wave) {
    if (row < a.len)
      for (int j = 0; j < k; ++j) {
        const double2 v = sm.Y[j * SS_LD + row];
        if (a.side == 1)
          left(row, j, v);
        else
          right(row, j, conj(v));
      }
  } else {
    small_project(sm, a.len, a.cnt, k, scale, tid, load, [&](int m, int c, double2 v) {
      if (a.side == 1)
        right(c, m, v);
      else
        left(c, m, conj(v));
    });
  }
}

// CholeskyQR of a small matrix in one launch, for centre moves: the general
// path's Gram, Cholesky panel (a 64-column one, 31 us), inverse, products,
// clears and copies are about sixteen launches.
// Elimination on [G | I] by the whole workgroup, one barrier a pivot: the row
// operations that turn G into R turn I into R^{-H}, both up to a row scale.
// Bound: the chain of pivots and the launch itself.  Measured: the exact
// 12-qubit build, with 96 moves, 23.7 -> 17.7 ms.
template <int N>
__global__ __launch_bounds__(SS_THREADS) void k_qr_small(QrSmallArgs a) {
  using D = SmallDims<N>;
  __shared__ SmallLds<N> sm;
  const int tid = threadIdx.x, row = tid - JSOLVE;
  const bool row_wave = tid >= JSOLVE;
  double2* G = sm.sv.G;
  double2* B = &sm.sv.B[0][0][0];   // N x N, ld 32
  static_assert(sizeof(sm.sv.B) >= 32 * 32 * sizeof(double2), "B in place of the solve's blocks");
  unsigned long long* dev = reinterpret_cast<unsigned long long*>(&sm.key[0]);
  const double sgn = a.x.conj ? -1.0 : 1.0;
  const auto load = [&](int r, int c) {
    const double2 v = *a.x.at(r, c);
    return make_double2(v.x, sgn * v.y);
  };
  if (row_wave) {
    const int lrow = min(row, a.len - 1);
#pragma unroll
    for (int c = 0; c < D::cols; ++c) {
      const double2 v = load(lrow, min(c, a.cnt - 1));
      sm.Y[c * SS_LD + row] = c < a.cnt && row < a.len ? v : make_double2(0.0, 0.0);
    }
  } else {
    for (int e = tid; e < 32 * N; e += JSOLVE) B[e] = make_double2((e >> 5) == (e & 31) ? 1.0 : 0.0, 0.0);
    if (tid == 0) *dev = 0;
  }
  __syncthreads();
  small_gram(sm, a.len, tid);
  bool ok = true;
  for (int k = 0; k < a.cnt; ++k) {
    const double d = G[33 * k].x;           // the same value in every thread: nobody writes row k any more
    if (!(d > 0.0) || !(d < 1e300)) {
      ok = false;
      break;
    }
    const double inv = 1.0 / d;
    for (int e = tid; e < (a.cnt - 1 - k) * 2 * N; e += SS_THREADS) {
      const int i = k + 1 + e / (2 * N), c = e & (2 * N - 1);
      double2* M = c < N ? G : B;
      const int j = c & (N - 1);
      const double2 f = G[k * 32 + i], r = M[k * 32 + j];
      double2& v = M[i * 32 + j];
      if (c >= N || j > k) {   // v -= conj(f) r / d
        const double fx = f.x * inv, fy = f.y * inv;
        v = make_double2(v.x - (fx * r.x + fy * r.y), v.y - (fx * r.y - fy * r.x));
      }
    }
    __syncthreads();
  }
  if (ok) {
    // R^{-1}[j][k] = conj(R^{-H}[k][j]), row k of R^{-H} = B's over sqrt(d_k)
    constexpr int GP = (32 * D::cols + SS_THREADS - 1) / SS_THREADS;
    double2 g[GP];
#pragma unroll
    for (int v = 0; v < GP; ++v) {
      const int e = tid + SS_THREADS * v, j = e >> 5, k = e & 31;
      const bool in = j < a.cnt && k < a.cnt;
      const double s = in ? 1.0 / sqrt(G[33 * k].x) : 0.0;
      const double2 b = in ? B[k * 32 + j] : make_double2(0.0, 0.0);
      g[v] = make_double2(b.x * s, -b.y * s);
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < GP; ++v)
      if (tid + SS_THREADS * v < 32 * D::cols) G[tid + SS_THREADS * v] = g[v];
    __syncthreads();
    small_apply(sm, a.len, tid);
    int steps = 3;
    for (int it = 0; it < steps && ok; ++it) {
      small_gram(sm, a.len, tid);
      if (it == 0) {
        double m = 0.0;
        for (int e = tid; e < 32 * a.cnt; e += SS_THREADS) {
          const int i = e >> 5, j = e & 31;
          if (j < a.cnt) {
            const double2 h = G[e];
            m = fmax(m, fmax(fabs(h.x - (i == j ? 1.0 : 0.0)), fabs(h.y)));
            if (!(h.x == h.x) || !(h.y == h.y)) m = 1e300;
          }
        }
        atomicMax(dev, (unsigned long long)__double_as_longlong(m));
        __syncthreads();
        const double defect = __longlong_as_double((long long)*dev);   // max |I - Q^H Q|
        ok = defect <= a.defect_max;
        steps = ns_steps_for(defect * a.cnt);
      }
      if (ok) {
        small_ns(sm, tid);
        small_apply(sm, a.len, tid);
      }
    }
  }
  if (tid == 0) *a.ok = ok ? 1 : 0;
  if (!ok) return;
  if (!row_wave)
    small_project(sm, a.len, a.cnt, a.cnt, 1.0, tid, load,
                  [&](int m, int c, double2 v) { a.p[(int64_t)m * a.cnt + c] = v; });
  __syncthreads();   // x is read; Q takes its place
  if (row_wave && row < a.len)
    for (int j = 0; j < a.cnt; ++j) {
      const double2 v = sm.Y[j * SS_LD + row];
      *a.x.at(row, j) = make_double2(v.x, sgn * v.y);
    }
}

void split_small(const SplitSmallArgs& a, hipStream_t s) {
  RCS_REQUIRE(a.len >= 1 && a.cnt >= 1 && split_small_fits(a.len, a.cnt) && a.ldx >= a.len && a.cap >= 1,
              "matrix too large for the small split");
  const dim3 grid(1), block(SS_THREADS);
  if (a.cnt <= 8)
    RCS_PROBED_LAUNCH(kKcFactor, k_split_small<8>, grid, block, 0, s, a);
  else if (a.cnt <= 16)
    RCS_PROBED_LAUNCH(kKcFactor, k_split_small<16>, grid, block, 0, s, a);
  else
    RCS_PROBED_LAUNCH(kKcFactor, k_split_small<32>, grid, block, 0, s, a);
  HIP_LAUNCH_OK();
}

void qr_small(const QrSmallArgs& a, hipStream_t s) {
  RCS_REQUIRE(a.cnt >= 1 && a.cnt <= a.len && split_small_fits(a.len, a.cnt) && a.len <= 2 * a.x.h,
              "matrix too large for the small QR");
  const dim3 grid(1), block(SS_THREADS);
  if (a.cnt <= 8)
    RCS_PROBED_LAUNCH(kKcFactor, k_qr_small<8>, grid, block, 0, s, a);
  else if (a.cnt <= 16)
    RCS_PROBED_LAUNCH(kKcFactor, k_qr_small<16>, grid, block, 0, s, a);
  else
    RCS_PROBED_LAUNCH(kKcFactor, k_qr_small<32>, grid, block, 0, s, a);
  HIP_LAUNCH_OK();
}

}  // namespace rcs
