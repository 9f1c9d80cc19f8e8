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

struct SplitSmallArgs {
  const double2* x;   // len x cnt, column-major, leading dimension ldx
  int ldx, len, cnt, cap;
  double eps;
  double tol, qtol;   // Jacobi tolerance and quadratic-stop level (0: off)
  double delta2;      // squared column norms below delta2 ||x||_F^2 count as zero
  int max_sweeps;
  int ns_steps;       // Newton-Schulz steps on the kept columns
  int sort, renorm;
  double2* wn;        // out: k orthonormal columns, ld ldx
  double2* p;         // out: k x cnt, row-major: wn^H x (/ nrm with renorm)
  double* sorted;     // out: cnt singular values, descending
  RankOut* out;
};
void split_small(const SplitSmallArgs& a, hipStream_t s);

// X = Q P of a small matrix, cnt <= len, by CholeskyQR with one to three
// Newton-Schulz steps; *ok = 0, and nothing else written, when a pivot is not
// positive or Q_1's orthogonality defect exceeds defect_max.
struct QrSmallArgs {
  const double2* x;   // len x cnt, column-major, leading dimension ldx
  int ldx, len, cnt;
  double defect_max;
  double2* wn;        // out: Q, ld ldx
  double2* p;         // out: cnt x cnt, row-major
  int* ok;
};
void qr_small(const QrSmallArgs& a, hipStream_t s);
// Newton-Schulz steps that take an orthogonality defect bounded by e to
// rounding (e -> 3 e^2 / 4 each).
__host__ __device__ inline int ns_steps_for(double e) { return e <= 1e-8 ? 1 : e <= 1e-4 ? 2 : 3; }

}  // namespace rcs
