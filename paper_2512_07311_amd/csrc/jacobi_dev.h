// Device code of the fp64 Jacobi rotations shared by the block Jacobi and the
// small split: per-precision types, plane rotations, inner schedules, the
// two-sided solve of a Gram in LDS and its application to rows held in
// registers.
#pragma once

#include <utility>

#include "common.h"

namespace rcs {

// Per-precision pieces: the complex type, the 16x16x4 matrix-core product
// and the row of accumulator element r in a lane (the fp64 instruction
// interleaves rows, the fp32 one gives each 16-lane group four consecutive
// rows).
template <typename R>
struct JT;
template <>
struct JT<double> {
  using C = double2;
  using V4 = double4_t;
  static constexpr double u = 1.11e-16;
  static constexpr double tiny = 1e-300;
  __device__ static V4 mma(double a, double b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int orow(int lane, int r) { return (lane >> 4) + 4 * r; }
  __host__ __device__ static C mk(double x, double y) { return make_double2(x, y); }
};
template <>
struct JT<float> {
  using C = float2;
  using V4 = float4_t;
  static constexpr double u = 5.97e-8;
  static constexpr float tiny = 1e-36f;
  __device__ static V4 mma(float a, float b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int orow(int lane, int r) { return 4 * (lane >> 4) + r; }
  __host__ __device__ static C mk(float x, float y) { return make_float2(x, y); }
};

// Plane rotation J = [[c, s e], [-s conj(e), c]] (rows: old columns i < j,
// columns: new) that (nearly) zeroes G_ij of the Hermitian 2x2 [[gii, g],
// [conj g, gjj]] in J^H G J; the identity when the pair is already
// orthogonal to tol or either column is negligible.
//
// Only unitarity has to hold to fp64 accuracy: the angle may be a few
// 1e-8 off (it leaves an off-diagonal of that relative size, which the
// next sweep's fresh Gram sees and removes, so convergence stays
// quadratic).  Hence e = g * rsq(|g|^2) with the raw hardware estimate
// (exact phase, modulus within ~2^-23 of one), tan(theta) in fp32 from
// tau = (gjj - gii) / (2|g|) (the smaller-angle root, |t| <= 1), and
// c = 1/sqrt(1 + t^2 |e|^2) refined in fp64, s = t c, which makes
// c^2 + s^2 |e|^2 = 1 to rounding.  Branch-free: inactive pairs select the
// identity.
template <typename R>
struct Rot {
  R c, s, ex, ey;
};
template <typename R>
__device__ inline bool rot_active(R gii, R gjj, R h2, R tol, R neg2) {
  return (gii > neg2) & (gjj > neg2) & (h2 > JT<R>::tiny) & (h2 > tol * tol * gii * gjj);
}
__device__ inline Rot<double> jac_rot(double gii, double gjj, double2 g, double tol, double neg2) {
  const double h2 = g.x * g.x + g.y * g.y;
  const bool act = rot_active<double>(gii, gjj, h2, tol, neg2);
  const double rh = __builtin_amdgcn_rsq(fmax(h2, 1e-300));
  const double tau = (gjj - gii) * (0.5 * rh);
  const float tf = (float)fabs(tau);
  const float root = tf + __builtin_amdgcn_sqrtf(fmaf(tf, tf, 1.0f));
  const float t32 = __builtin_amdgcn_rcpf(tf > 1e18f ? 2.0f * tf : root);
  const double t = tau < 0.0 ? -(double)t32 : (double)t32;
  const double ex = g.x * rh, ey = g.y * rh;
  const double c = rsqrt_fast(fma(t * t, ex * ex + ey * ey, 1.0));
  Rot<double> r;
  r.c = act ? c : 1.0;
  r.s = act ? t * c : 0.0;
  r.ex = act ? ex : 1.0;
  r.ey = act ? ey : 0.0;
  return r;
}

// fp32: the same rotation with every step in fp32; c takes one Newton step
// on the hardware 1/sqrt estimate, so c^2 (1 + t^2 |e|^2) = 1 to fp32
// rounding.
__device__ inline Rot<float> jac_rot(float gii, float gjj, float2 g, float tol, float neg2) {
  const float h2 = g.x * g.x + g.y * g.y;
  const bool act = rot_active<float>(gii, gjj, h2, tol, neg2);
  const float rh = __builtin_amdgcn_rsqf(fmaxf(h2, JT<float>::tiny));
  const float tau = (gjj - gii) * (0.5f * rh);
  const float tf = fabsf(tau);
  const float root = tf + __builtin_amdgcn_sqrtf(fmaf(tf, tf, 1.0f));
  const float t32 = __builtin_amdgcn_rcpf(tf > 1e18f ? 2.0f * tf : root);
  const float t = tau < 0.0f ? -t32 : t32;
  const float ex = g.x * rh, ey = g.y * rh;
  const float x = fmaf(t * t, ex * ex + ey * ey, 1.0f);
  float c = __builtin_amdgcn_rsqf(x);
  c = fmaf(c, fmaf(-0.5f * x * c, c, 0.5f), c);
  Rot<float> r;
  r.c = act ? c : 1.0f;
  r.s = act ? t * c : 0.0f;
  r.ex = act ? ex : 1.0f;
  r.ey = act ? ey : 0.0f;
  return r;
}

// With a = s e (precomputed once per rotation: RotA = {c, Re a, Im a}):
// right action (X J):  x_i' = c x_i - conj(a) x_j,  x_j' = a x_i + c x_j;
// left action (J^H X): x_i' = c x_i - a x_j,        x_j' = conj(a) x_i + c x_j.
template <typename R>
struct RotA {
  R c, ax, ay;
};
template <typename R>
__device__ inline RotA<R> rot_a(const Rot<R>& r) { return RotA<R>{r.c, r.s * r.ex, r.s * r.ey}; }
template <typename R, typename C>
__device__ inline void rot_right(const RotA<R>& r, C& xi, C& xj) {
  const R ax = r.ax, ay = r.ay;
  const C ni(fma(r.c, xi.x, -fma(ax, xj.x, ay * xj.y)), fma(r.c, xi.y, fma(ay, xj.x, -ax * xj.y)));
  xj = C(fma(r.c, xj.x, fma(ax, xi.x, -ay * xi.y)), fma(r.c, xj.y, fma(ax, xi.y, ay * xi.x)));
  xi = ni;
}
template <typename R, typename C>
__device__ inline void rot_left(const RotA<R>& r, C& xi, C& xj) {
  const R ax = r.ax, ay = r.ay;
  const C ni(fma(r.c, xi.x, -fma(ax, xj.x, -ay * xj.y)), fma(r.c, xi.y, -fma(ax, xj.y, ay * xj.x)));
  xj = C(fma(r.c, xj.x, fma(ax, xi.x, ay * xi.y)), fma(r.c, xj.y, fma(ax, xi.y, -ay * xi.x)));
  xi = ni;
}

// ------------------------------------------------- row-resident rotation
// The fp64 rotate pass for 16-column blocks.  The two-sided solve of the
// 32 x 32 Gram is a serial chain of rounds (16 disjoint rotations each), and
// forming the unitary and multiplying by it costs twice the flops of
// applying the rotations themselves, at the same fp64 rate (the vector and
// the matrix units both reach 78.6 TFLOP/s).  So the workgroup splits:
//   waves 0-2   run the solve, one barrier per round: thread (k, b) holds the
//               block of pair a = b + k mod 16 against pair b, computes pair
//               b's rotation itself, takes pair a's from the lane that has
//               it, and moves its four entries to where the next round needs
//               them;
//   wave 3      computes the same 16 rotations, one a lane, and publishes
//               them in the form the row waves want;
//   waves 4...  hold one row of Y_p per lane in registers (32 columns, loaded
//               while the partial Grams are summed) and apply each round's
//               rotations one round behind the solve.
// A rotation is applied as two in-place complex shears with the column scales
// deferred (an LDU factorisation of the plane rotation, eight FMAs instead of
// twelve):  with x = d x~,  x~_i -= conj(u) x~_j,  x~_j += w x~_i',
//   u = t d_j / d_i,  w = c^2 t d_i / d_j,  d_i <- c d_i,  d_j <- d_j / c,
// t the complex tangent (|t| <= 1), c = (1 + |t|^2)^(-1/2).  The scales stay
// within 2^(+-rounds / 2) and are multiplied out before the rows are stored.
// Rotation q sits in lane q of every 16-lane row, from where the FMA itself
// broadcasts it (DPP row_newbcast, the one DPP form 64-bit operations have):
// 5.6 cycles per FMA and wave, against 7.2 with separate moves (plain: 4.9).
//
// Bound: below about 1024 columns the chain of rounds (0.48 us each: reads
// 200 cycles, rotation 210, exchange 140, 4 x 12 fp64 operations 300, writes
// and barrier 300), at 2048 the fp64 vector rate (two row waves and one solver
// wave per SIMD) and the read and write of the matrix (64 MB, 25 us on its
// own).  Measured, per launch at 64 x 64 / 512 x 512: the LDS solve with a V
// product on the matrix cores (still the 32-column and fp32 form) 21.5 / 22
// us, this scheme 12.1 / 13.7 us; 2048 x 2048 43 -> 32 us inside an SVD (28
// since the Gram pass leaves it a quarter of the partials).  Its
// first form, a full Gram of 256 blocks in four waves, places computed each
// round and the shears from a row wave, took 15.2 / 16.7 us: index arithmetic
// between barriers cost 310 cycles a round.  Tried and slower: the whole
// solve before any row work (41 us at 2048), a rolled row loop with register
// rotation.
constexpr int JSOLVE = 256;   // threads of waves 0-3

// Inner schedules: pair q of round r is columns i(q, r) and j(q, r).
//   SchedRR<N>  : round robin over N columns, N/2 pairs, N - 1 rounds;
//   SchedCross  : two 16-column blocks against each other, 16 rounds;
//   SchedFull   : the round robin inside both blocks at once, then the cross
//                 rounds: every pair of the 32 columns once.
// Slot s of a round is pair s's first column, slot pairs + s its second one.
// Between rounds the columns move by a fixed permutation of the slots, next(),
// per segment of rounds; after the last segment they are back where they began.
template <int N>
struct SchedRR {
  static constexpr int cols = N, pairs = N / 2, rounds = N - 1, segments = 1;
  __host__ __device__ static constexpr int i(int q, int r) { return q == 0 ? 0 : ((q - 1 + r) % (N - 1)) + 1; }
  __host__ __device__ static constexpr int j(int q, int r) { return ((N - 2 - q + r) % (N - 1)) + 1; }
  __host__ __device__ static constexpr int segment(int) { return rounds; }
  // column 0 stays; column ((x + r) mod (N - 1)) + 1 is at place x of a ring
  __host__ __device__ static constexpr int ring(int s) { return s < pairs ? s - 1 : N - 2 - (s - pairs); }
  __host__ __device__ static constexpr int unring(int x) { return x <= pairs - 2 ? x + 1 : pairs + N - 2 - x; }
  __host__ __device__ static constexpr int next(int s, int) {
    return s == 0 ? 0 : unring(ring(s) == 0 ? N - 2 : ring(s) - 1);
  }
};
struct SchedCross {
  static constexpr int cols = 32, pairs = 16, rounds = 16, segments = 1;
  __host__ __device__ static constexpr int i(int q, int) { return q; }
  __host__ __device__ static constexpr int j(int q, int r) { return 16 + ((q + r) & 15); }
  __host__ __device__ static constexpr int segment(int) { return rounds; }
  __host__ __device__ static constexpr int next(int s, int) { return s < 16 ? s : 16 + ((s - 1) & 15); }
};
struct SchedFull {
  using RR = SchedRR<16>;
  static constexpr int cols = 32, pairs = 16, rounds = 31, segments = 4;
  __host__ __device__ static constexpr int i(int q, int r) { return r < 15 ? (q & 8) * 2 + RR::i(q & 7, r) : q; }
  __host__ __device__ static constexpr int j(int q, int r) {
    return r < 15 ? (q & 8) * 2 + RR::j(q & 7, r) : SchedCross::j(q, r - 15);
  }
  // 14 steps of the round robins, one from their end to the cross rounds, 15
  // steps of these, one back
  __host__ __device__ static constexpr int segment(int g) { return g == 0 ? 14 : g == 2 ? 15 : 1; }
  __host__ __device__ static constexpr int next(int s, int g) {
    if (g < 2) {
      const int half = s & 8, t = RR::next((s & 7) | (s & 16) >> 1, 0);   // slot within the block's round robin
      if (g == 0) return half | (t & 7) | (t & 8) << 1;
      return half * 2 + (t < 8 ? RR::i(t, 0) : RR::j(t - 8, 0));           // cross slots are the columns
    }
    const int c = SchedCross::next(s, 0);
    if (g == 2) return c;
    const int t = (c & 15) == 0 ? 0 : RR::unring((c & 15) - 1);
    return (c & 16) >> 1 | (t & 7) | (t & 8) << 1;
  }
};

// a_k -= conj(u_k) b_k resp. a_k += w_k b_k for four independent columns k,
// u_k, w_k taken from lane Q + k of the 16-lane row.  Four at a time, so that
// dependent FMAs are eight instructions apart (two apart they cost twice the
// time with one row wave per SIMD).  The leading wait covers a u or w that
// the compiler moved with a VALU instruction just before (a DPP source needs
// two wait states after one).
template <int Q>
__device__ __forceinline__ void shear_sub(double2& a0, double2& a1, double2& a2, double2& a3, const double2& b0,
                                          const double2& b1, const double2& b2, const double2& b3, const double2& u) {
  asm(
      "s_nop 1\n\t"
      "v_fmac_f64_dpp %0, -%16, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, -%16, %10 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, -%16, %12 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, -%16, %14 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, -%16, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, -%16, %11 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, -%16, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, -%16, %15 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, -%17, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, -%17, %11 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, -%17, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, -%17, %15 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %17, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %17, %10 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %17, %12 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %17, %14 row_newbcast:%21 row_mask:0xf bank_mask:0xf"
      : "+v"(a0.x), "+v"(a0.y), "+v"(a1.x), "+v"(a1.y), "+v"(a2.x), "+v"(a2.y), "+v"(a3.x), "+v"(a3.y)
      : "v"(b0.x), "v"(b0.y), "v"(b1.x), "v"(b1.y), "v"(b2.x), "v"(b2.y), "v"(b3.x), "v"(b3.y), "v"(u.x), "v"(u.y),
        "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3));
}
template <int Q>
__device__ __forceinline__ void shear_add(double2& a0, double2& a1, double2& a2, double2& a3, const double2& b0,
                                          const double2& b1, const double2& b2, const double2& b3, const double2& w) {
  asm(
      "s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %16, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %16, %10 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, %16, %12 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, %16, %14 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %16, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %16, %11 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %16, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %16, %15 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, -%17, %9 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, -%17, %11 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %4, -%17, %13 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %6, -%17, %15 row_newbcast:%21 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %17, %8 row_newbcast:%18 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %17, %10 row_newbcast:%19 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %5, %17, %12 row_newbcast:%20 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %7, %17, %14 row_newbcast:%21 row_mask:0xf bank_mask:0xf"
      : "+v"(a0.x), "+v"(a0.y), "+v"(a1.x), "+v"(a1.y), "+v"(a2.x), "+v"(a2.y), "+v"(a3.x), "+v"(a3.y)
      : "v"(b0.x), "v"(b0.y), "v"(b1.x), "v"(b1.y), "v"(b2.x), "v"(b2.y), "v"(b3.x), "v"(b3.y), "v"(w.x), "v"(w.y),
        "n"(Q), "n"(Q + 1), "n"(Q + 2), "n"(Q + 3));
}

// Round r's rotations on a row.
template <class S, int R_, int Q>
__device__ __forceinline__ void apply_four(double2 (&y)[S::cols], const double2& u, const double2& w) {
  constexpr int i0 = S::i(Q, R_), i1 = S::i(Q + 1, R_), i2 = S::i(Q + 2, R_), i3 = S::i(Q + 3, R_);
  constexpr int j0 = S::j(Q, R_), j1 = S::j(Q + 1, R_), j2 = S::j(Q + 2, R_), j3 = S::j(Q + 3, R_);
  shear_sub<Q>(y[i0], y[i1], y[i2], y[i3], y[j0], y[j1], y[j2], y[j3], u);
  shear_add<Q>(y[j0], y[j1], y[j2], y[j3], y[i0], y[i1], y[i2], y[i3], w);
}
template <class S, int R_>
__device__ __forceinline__ void apply_round(double2 (&y)[S::cols], const double2& u, const double2& w) {
  apply_four<S, R_, 0>(y, u, w);
  if constexpr (S::pairs > 4) apply_four<S, R_, 4>(y, u, w);
  if constexpr (S::pairs > 8) {
    apply_four<S, R_, 8>(y, u, w);
    apply_four<S, R_, 12>(y, u, w);
  }
}

// The rotation of jac_rot in the form the row-resident pass wants: c and
// a = c t with t = +-g / (|d| + sqrt(d^2 + |g|^2)), d = (gjj - gii) / 2 (the
// smaller-angle root), and 1 / c.  t may be off by the hardware estimates'
// ~1e-8 (see jac_rot); c is refined, so c^2 (1 + |t|^2) = 1 to rounding.
// Range: d^2 and |g|^2 have to stay finite and, for pairs that rotate, well
// above the guard of 1e-300: jacobi_run scales columns whose summed squares are
// not within 2^(+-300), and the small split's matrices have unit norm.
// The dependent chain is what a round waits
// for: the guard against 0 sits in |g|^2's first product, an inactive pair's
// infinity in the addend of the denominator, the sign on g, and the test is
// one comparison (a conjunction of four goes through the scalar unit).
struct RotT {
  double c, ax, ay, ci, x;   // x: 1 + |t|^2
};
__device__ inline RotT jac_rot_t(double gii, double gjj, double2 g, double tol, double neg2) {
  const double h2 = fma(g.x, g.x, fma(g.y, g.y, 1e-300)), d = 0.5 * (gjj - gii);
  const double lim = (gii < gjj ? gii : gjj) > neg2 ? tol * tol * (gii * gjj) : __builtin_inf();
  const double m = h2 > fmax(lim, JT<double>::tiny) ? fabs(d) : __builtin_inf();
  const double s = fma(d, d, h2);
  const double k = __builtin_amdgcn_rcp(fma(s, __builtin_amdgcn_rsq(s), m));
  const double x = fma(k * k, h2, 1.0);
  // 1/sqrt(x), x in [1, 2]: the estimate's relative error e goes to e^3
  const double q = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * q, q, 1.0);
  RotT r;
  r.c = fma(q * e, fma(0.375, e, 0.5), q);
  r.ci = x * r.c;
  r.x = x;
  const double ct = r.c * k;
  r.ax = (d < 0.0 ? -g.x : g.x) * ct;
  r.ay = (d < 0.0 ? -g.y : g.y) * ct;
  return r;
}

struct SolveLds {
  double2 G[32 * 32];      // the Gram, all of it
  double2 B[2][4][192];    // the solve's copy: entry (side a, side b) of a thread's pair block
  double2 rot[2][2][16];   // u and w of a round's rotations, from the publishing wave
  double scale[32], scale_err[32];   // column scales are scale (1 + scale_err)
  unsigned short pair[31][16];   // the schedule: i | j << 8
  int any_flag, big;
};

__device__ __forceinline__ double column_scale(const SolveLds& sm, int c) {
  return fma(sm.scale[c], sm.scale_err[c], sm.scale[c]);
}

// Round r's shears on the lane's row.
template <class S, int R_>
__device__ __forceinline__ void apply_published(double2 (&y)[S::cols], const SolveLds& sm, int buf, int lane) {
  const double2 u = sm.rot[buf][0][lane & 15], w = sm.rot[buf][1][lane & 15];
  apply_round<S, R_>(y, u, w);
}

// While the solve is at round r, every row wave applies round r - 1 (the last
// round of the previous inner sweep, if any, for r = 0).
template <class S, int R_>
__device__ __forceinline__ void row_phase(double2 (&y)[S::cols], const SolveLds& sm, int& buf, int lane,
                                          bool pending) {
  constexpr int P = (R_ + S::rounds - 1) % S::rounds;
  if (R_ > 0 || pending) apply_published<S, P>(y, sm, buf ^ 1, lane);
  __syncthreads();
  buf ^= 1;
}
template <class S, int... R_>
__device__ __forceinline__ void row_phases(double2 (&y)[S::cols], const SolveLds& sm, int& buf, int lane, bool pending,
                                           std::integer_sequence<int, R_...>) {
  (row_phase<S, R_>(y, sm, buf, lane, pending), ...);
}
// The row waves' side of `inner` sweeps (inner * rounds barriers); the rows
// are left with their column scales in sm.scale.
template <class S>
__device__ __forceinline__ void row_sweeps(double2 (&y)[S::cols], const SolveLds& sm, int lane, int inner) {
  int buf = 0;
  for (int in = 0; in < inner; ++in)
    row_phases<S>(y, sm, buf, lane, in > 0, std::make_integer_sequence<int, S::rounds>{});
  apply_published<S, S::rounds - 1>(y, sm, buf ^ 1, lane);
}

// The schedule's pairs, for the solve (all of `nthreads` threads).
template <class S>
__device__ inline void fill_schedule(SolveLds& sm, int tid, int nthreads) {
  for (int e = tid; e < S::rounds * 16; e += nthreads) {
    const int q = e & 15, r = e >> 4;
    if (q < S::pairs) sm.pair[r][q] = (unsigned short)(S::i(q, r) | S::j(q, r) << 8);
  }
}

// The solve.  Thread (k, b) = tid = k P + b, k <= P / 2, has the 2 x 2 block of
// pair a = b + k mod P against pair b: the Gram is Hermitian, so each block
// of two pairs is kept once, at its thread's own place.  As the columns move
// between rounds by a fixed permutation of the slots, so do the entries
// between the threads' places: a thread reads its block from one place and
// writes its entries to four others in every round, with no index arithmetic
// between barriers (which cost more there than the rotation itself).
template <class S>
struct Blocks {
  static constexpr int P = S::pairs, n = P * P / 2 + P / 2, waves = (P * P / 2 + P + 63) / 64;
};
// Place of entry (slot sa, slot sb), a byte offset into B[.], with the sign
// bit set where the place holds its conjugate.
template <class S>
__device__ inline unsigned block_entry(int sa, int sb) {
  constexpr int P = S::pairs;
  const int qa = sa & (P - 1), qb = sb & (P - 1), ha = sa / P, hb = sb / P;
  const int k = (qa - qb) & (P - 1);
  const bool swap = k > P / 2 || (k == P / 2 && qb >= P / 2) || (k == 0 && ha > hb);
  const int at = swap ? ((P - k) & (P - 1)) * P + qa : k * P + qb;
  const int type = swap ? 2 * hb + ha : 2 * ha + hb;
  return (unsigned)((type * 192 + at) * (int)sizeof(double2)) | (swap ? 0x80000000u : 0u);
}
// Thread tid's block from the Gram (all solver threads; a barrier follows).
template <class S>
__device__ inline void load_blocks(SolveLds& sm, int tid) {
  constexpr int P = S::pairs;
  if (tid >= Blocks<S>::waves * 64) return;
  const int qb = tid & (P - 1), qa = (qb + tid / P) & (P - 1);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int row = t >= 2 ? S::j(qa, 0) : S::i(qa, 0), col = t & 1 ? S::j(qb, 0) : S::i(qb, 0);
    sm.B[0][t][tid] = sm.G[row * 32 + col];
  }
}
__device__ __forceinline__ void block_write(SolveLds& sm, int buf, unsigned e, double2 v) {
  v.y = __hiloint2double(__double2hiint(v.y) ^ (int)(e & 0x80000000u), __double2loint(v.y));
  *reinterpret_cast<double2*>(reinterpret_cast<char*>(&sm.B[0][0][0]) +
                              (buf * (int)sizeof(sm.B[0]) + (int)(e & 0x7fffu))) = v;
}

// Where thread tid's entries go, by segment.  The last wave's spare lanes work
// on places of their own.
template <class S>
struct Moves {
  unsigned e[S::segments][4];
};
template <class S>
__device__ inline Moves<S> block_moves(int tid) {
  constexpr int P = S::pairs;
  const int qb = tid & (P - 1), qa = (qb + tid / P) & (P - 1);
  Moves<S> m;
#pragma unroll
  for (int g = 0; g < S::segments; ++g) {
    const int ia = S::next(qa, g), ja = S::next(qa + P, g), ib = S::next(qb, g), jb = S::next(qb + P, g);
    const int to[4][2] = {{ia, ib}, {ia, jb}, {ja, ib}, {ja, jb}};
#pragma unroll
    for (int t = 0; t < 4; ++t)
      m.e[g][t] = tid < Blocks<S>::n ? block_entry<S>(to[t][0], to[t][1])
                                     : (unsigned)((t * 192 + min(tid, 191)) * (int)sizeof(double2));
  }
  return m;
}

// The publishing wave's side: it takes the same rotations from the blocks as
// the solve does, one a lane, and turns them into shears with the column
// scales, which the solve's chain does not wait for.
// The rounding of c, 1 / c and the scales is the same for a whole column, so it
// does not average out in the column's norm as that of its entries does: what
// it was is added up per column, a round behind.  Singular values, relative to
// 64-bit ones, geometric mean over 40 matrices of up to about 1,000 columns:
// 0.06 of the error without it, 0.07 of that of a product with the unitary.  SVD
// 203 x 131 and 2048 x 2048 take 2.17 and 80.6 ms without, 2.14 and 80.9 with
// (two runs differ by 4% and 0.4%).
template <class S>
__device__ inline void publish_sweeps(SolveLds& sm, int lane, double tol_in, double neg2, int inner) {
  constexpr int P = S::pairs;
  const int q = lane & (P - 1);
  int buf = 0, li = q, lj = P + q;   // the previous round's columns and
  double pi = 0.0, pj = 0.0;         // errors of their scales
  auto add_err = [&] {
    if (lane < P) {
      sm.scale_err[li] += pi;
      sm.scale_err[lj] += pj;
    }
  };
  for (int left = inner * S::rounds, r = 0; left > 0; --left) {
    const double gii = sm.B[buf][0][q].x, gjj = sm.B[buf][3][q].x;
    const double2 gij = sm.B[buf][1][q];
    const int pair = sm.pair[r][q], i = pair & 31, j = pair >> 8;
    add_err();
    const double di = sm.scale[i], dj = sm.scale[j];
    const double ri = rcp_fast(di), rj = rcp_fast(dj);
    const double qi = dj * ri, qj = di * rj;
    const RotT t = jac_rot_t(gii, gjj, gij, tol_in, neg2);
    const double ni = di * t.c, nj = dj * t.ci;
    if (lane < P) {
      const double fu = t.ci * qi, fw = t.c * qj;
      sm.rot[buf][0][q] = make_double2(t.ax * fu, t.ay * fu);
      sm.rot[buf][1][q] = make_double2(t.ax * fw, t.ay * fw);
      sm.scale[i] = ni;
      sm.scale[j] = nj;
    }
    // x c = ci (1 + rc), x c^2 = 1 + 2 ec, di c = ni + ..., dj ci = nj + ...
    const double rc = fma(t.x, t.c, -t.ci) * t.c, ec = 0.5 * (fma(t.ci, t.c, -1.0) + rc);
    pi = fma(di, t.c, -ni) * ri - ec;
    pj = fma(dj, t.ci, -nj) * rj + (rc - ec);
    li = i;
    lj = j;
    if (left == 1) add_err();
    __syncthreads();
    buf ^= 1;
    r = r + 1 == S::rounds ? 0 : r + 1;
  }
}

// The first JSOLVE threads' side: `inner` sweeps of two-sided rotations on
// the blocks in B[0] by waves 0-2, publishing by wave 3.
template <class S>
__device__ inline void solve_sweeps(SolveLds& sm, const Moves<S>& mv, int tid, double tol_in, double neg2,
                                    int inner) {
  constexpr int P = S::pairs;
  const int lane = tid & 63;
  if (tid >= JSOLVE - 64) {
    publish_sweeps<S>(sm, lane, tol_in, neg2, inner);
    return;
  }
  if (tid >= Blocks<S>::waves * 64) {   // whole waves with no block
    for (int left = inner * S::rounds; left > 0; --left) __syncthreads();
    return;
  }
  const int qb = tid & (P - 1), qa = (qb + tid / P) & (P - 1), lane_a = (lane & ~(P - 1)) + qa;
  int buf = 0;
  for (int in = 0; in < inner; ++in) {
#pragma unroll
    for (int g = 0; g < S::segments; ++g) {
      for (int left = S::segment(g); left > 0; --left) {
        const double gii = sm.B[buf][0][qb].x, gjj = sm.B[buf][3][qb].x;   // thread (0, b)'s block
        const double2 gij = sm.B[buf][1][qb];
        double2 g00 = sm.B[buf][0][tid], g01 = sm.B[buf][1][tid], g10 = sm.B[buf][2][tid], g11 = sm.B[buf][3][tid];
        __builtin_amdgcn_sched_barrier(0);   // all reads on their way before the rotation's chain
        const RotT t = jac_rot_t(gii, gjj, gij, tol_in, neg2);
        const RotA<double> rb{t.c, t.ax, t.ay};
        RotA<double> ra;
        ra.c = __shfl(rb.c, lane_a);
        ra.ax = __shfl(rb.ax, lane_a);
        ra.ay = __shfl(rb.ay, lane_a);
        if (tid < P) g10 = make_double2(gij.x, -gij.y);   // not kept
        rot_right(rb, g00, g01);
        rot_right(rb, g10, g11);
        rot_left(ra, g00, g10);
        rot_left(ra, g01, g11);
        buf ^= 1;
        block_write(sm, buf, mv.e[g][2], g10);
        block_write(sm, buf, mv.e[g][0], g00);
        block_write(sm, buf, mv.e[g][1], g01);   // k = 0: to g10's place
        block_write(sm, buf, mv.e[g][3], g11);
        __syncthreads();
      }
    }
  }
}

}  // namespace rcs
