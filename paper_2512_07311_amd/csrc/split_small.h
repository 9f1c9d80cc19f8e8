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

}  // namespace rcs
