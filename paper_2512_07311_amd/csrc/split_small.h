// Internal interface of the one-launch split of small two-site matrices.
#pragma once

#include "common.h"

namespace rcs {

// Result of the rank rule (build.hip, k_sort_rank).
struct RankOut {
  int k;
  int nnz;
  double eps_step, w, nrm;
  int bad;
  int sweeps;   // split_small only; -1: not converged
};

constexpr int kSplitSmallRows = 128, kSplitSmallCols = 32;
inline bool split_small_fits(int len, int cnt) { return len <= kSplitSmallRows && cnt <= kSplitSmallCols; }

// Where a small kernel's matrix lives: element (r, c) at
// p[(r / h) hs + (r % h) rs + c cs], conjugated if conj.  Covers both
// orientations of a site tensor [s][a][b] and plain columns.
struct MatView {
  double2* p;
  int64_t hs, rs, cs;
  int h, conj;
  __device__ inline double2* at(int r, int c) const {
    const int top = r >= h ? 1 : 0;   // at most two halves
    return p + top * hs + (int64_t)(r - top * h) * rs + c * cs;
  }
};

struct SplitSmallArgs {
  const double2* x;   // len x cnt, column-major, leading dimension ldx
  int ldx, len, cnt, cap;
  double eps;
  double tol, qtol;   // Jacobi tolerance and quadratic-stop level (0: off)
  double delta2;      // squared column norms below delta2 ||x||_F^2 count as zero
  int max_sweeps;
  int ns_steps;       // Newton-Schulz steps on the kept columns
  int sort, renorm;
  // Out, in this order of preference: the two factors straight into the sites
  // (ai, aj: tensors [s][dl][k] and [s][k][dr]; side 1: the rows of x are
  // ai's, side 2: conjugated, aj's), or, without sites, k orthonormal columns
  // wn (ld ldx) and p = wn^H x (k x cnt, row-major), over nrm with renorm.
  double2 *ai, *aj;
  int dl, dr, side;
  double2 *wn, *p;
  double* sorted;     // cnt singular values, descending
  RankOut* out;       // device or pinned host memory
};
void split_small(const SplitSmallArgs& a, hipStream_t s);

// X = Q P of a small matrix, cnt <= len, by CholeskyQR with one to three
// Newton-Schulz steps; *ok = 0, and nothing else written, when a pivot is not
// positive or Q_1's orthogonality defect exceeds defect_max.
struct QrSmallArgs {
  MatView x;          // len x cnt; replaced by Q
  int len, cnt;
  double defect_max;
  double2* p;         // out: cnt x cnt, row-major
  int* ok;            // device or pinned host memory
};
void qr_small(const QrSmallArgs& a, hipStream_t s);
// Newton-Schulz steps that take an orthogonality defect bounded by e to
// rounding (e -> 3 e^2 / 4 each).
__host__ __device__ inline int ns_steps_for(double e) { return e <= 1e-8 ? 1 : e <= 1e-4 ? 2 : 3; }

}  // namespace rcs
