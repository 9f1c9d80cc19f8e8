// Internal interface of the state builder.
#pragma once

#include <vector>

#include "circuit.h"
#include "state.h"

namespace rcs {

struct BuildOptions {
  int contraction = RCS_PREC_C128;
  int rank_mode = RCS_RANK_FULL_SVD;
  double fallback_tau = 1e-6;
  std::vector<float> mlp;
  int rsvd_p = 16, rsvd_q = 2;
  uint64_t rsvd_seed = 0;
  void* stream = nullptr;
  bool log_spectra = false;
  int max_ops = -1;
  bool canonicalize = true;
  bool svd_f32 = false;      // RCS_SVD_F32
};

struct BuildWork;
BuildWork* new_work();
void delete_work(BuildWork* w);

// Runs the schedule of circuit c on the freshly allocated state st.
void build_one(rcs_state_s& st, const rcs_circuit_s& c, int chi, double eps, const BuildOptions& o,
               BuildWork& ws);

// Learned-rank network pieces (fp32).
void spectrum_features(const double* s_dev, int k, int bond, int n_sites, int cycle, int n_cycles,
                       float* feat_dev, hipStream_t st);
void mlp_forward(const float* w, const float* x, int batch, float* out, hipStream_t s);

// A site tensor: element (s, a, b) at p[s * s_stride + a * ld + b].
struct SiteView {
  const double2* p;
  int64_t s;
  int ld;
};
struct Gate4 {
  double2 g[16];
};
// Where a two-site matrix goes, column-major with leading dimension ld.
// orient 1: M, rows (s1, a), columns (s2, c); orient 2: M^H.  x0: a second
// copy, or null.
struct MixOut {
  double2* x;
  double2* x0;
  int ld, orient;
};
// Entry (a, c) of theta' from its four products.
__device__ inline void mix_store(const double2 (&t)[4], const Gate4& G, int a, int c, int dl, int dr,
                                 const MixOut& out) {
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double2 g = G.g[o * 4 + q];
      re += g.x * t[q].x - g.y * t[q].y;
      im += g.x * t[q].y + g.y * t[q].x;
    }
    const int row = (o >> 1) * dl + a, col = (o & 1) * dr + c;
    const int64_t idx = out.orient == 1 ? (int64_t)col * out.ld + row : (int64_t)row * out.ld + col;
    const double2 v = make_double2(re, out.orient == 1 ? im : -im);
    out.x[idx] = v;
    if (out.x0) out.x0[idx] = v;
  }
}
// theta' of A (dl x dm per s) and B (dm x dr per s) in the given precision.
void contract_mix(const SiteView& A, const SiteView& B, const Gate4& G, int dl, int dm, int dr, int precision,
                  const MixOut& out, hipStream_t s);
// The same in complex64 or split bf16.
void contract_mix_lowp(const SiteView& A, const SiteView& B, const Gate4& G, int dl, int dm, int dr, int precision,
                       const MixOut& out, hipStream_t s, hipEvent_t start, hipEvent_t stop);

}  // namespace rcs
