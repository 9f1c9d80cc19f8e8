// Internal interface of the one-sided block Jacobi SVD (fp64 and fp32).
#pragma once

#include "common.h"

namespace rcs {

// Sweep limit of every SVD.  Flat spectra take 10 to 14 sweeps; an
// unpreconditioned matrix whose spectrum spans 12 decades takes about 60 at
// 4096 columns, so the limit stands well clear of that.
constexpr int kJacobiMaxSweeps = 120;

struct JacobiPlan {
  int jb = 16;            // columns per block (16 or 32)
  int inner = 1;          // inner sweeps per pair meeting
  int len = 0, cnt = 0;   // matrix is len x cnt
  int ldx = 0;            // leading dimension (rows, padded to 64)
  int nbp = 0;            // number of column blocks (even)
  int cnt_pad = 0;        // nbp * 32 columns allocated
  int n_pairs = 0;
  int n_chunks = 0, rows_per_chunk = 0;     // rotate pass row chunks
  int n_gchunks = 0, rows_per_gchunk = 0;   // Gram pass row chunks
};

// Tolerances of the fp64 iteration on len rows: relative orthogonality (tol >
// 0 replaces the default), the squared cosine below which the next sweep
// would rotate nothing (0: rule off), and the squared column norm, relative
// to ||X||_F^2, that counts as zero.
struct JacobiTol {
  double tol, qtol, delta2;
};
JacobiTol jacobi_tol(int len, double tol = 0.0);

// jb <= 0 picks the default block width for the shape; f32: the plan of
// jacobi_run_f32 (its Gram chunks differ).
JacobiPlan jacobi_plan(int len, int cnt, int jb = 0, bool f32 = false);
size_t jacobi_work_bytes(const JacobiPlan& pl);
// RCS_DEBUG_JACOBI=1: every SVD's sweeps on stderr.
bool jacobi_debug();
// Orthogonalises the columns of x in place; returns the number of sweeps
// (the last one rotates nothing, or its largest entering cosine squared is
// below tol / 100, after which the next would rotate nothing: quadratic
// convergence).  fro2 = ||x||_F^2; columns below
// 8 u sqrt(len) ||x||_F count as numerically zero.
// tol > 0 replaces the default relative orthogonality tolerance 16 u sqrt(len).
// rot_count_dev and rot_count_host hold two ints (rotation count; whether a
// meeting of the sweep entered with a squared cosine above tol / 100).
int jacobi_run(const JacobiPlan& pl, double2* x, void* work, int* rot_count_dev,
               int* rot_count_host, double fro2, hipStream_t stream, int max_sweeps, double tol = 0.0);
// The same in fp32 (complex64 columns, u = 2^-24); work as sized by
// jacobi_work_bytes.
int jacobi_run_f32(const JacobiPlan& pl, float2* x, void* work, int* rot_count_dev,
                   int* rot_count_host, double fro2, hipStream_t stream, int max_sweeps, double tol = 0.0);

}  // namespace rcs
