// Rank-prediction network and its training kernels (fp32).
//
// Network: Linear(66,128) - ReLU - Linear(128,128) - ReLU - Linear(128,32),
// packed weights W1[128][66], b1[128], W2[128][128], b2[128], W3[32][128],
// b3[32].  Loss: mean over batch and outputs of (out - y)^2.  Every
// reduction has a fixed order, so forward, backward and Adam are
// deterministic.
//
// Features (66): 64-bin histogram of log10(s^2 / sum s^2) of a bond's kept
// singular values (0.25-decade bins over [-16, 0), clamped at both ends,
// normalised to sum 1), then bond / (n - 2) and cycle / n_cycles.
#include "state.h"

namespace rcs {

constexpr int NI = 66, NH = 128, NO = 32;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NI, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NO * NH, N_PARAMS = OFF_B3 + NO;
static_assert(N_PARAMS == RCS_MLP_PARAMS, "parameter count");

// -------------------------------------------------------------- features
__global__ void k_spec_features(const double* s, int k, double bond_f, double cycle_f, float* feat) {
  __shared__ double red[256];
  __shared__ int hist[64];
  const int tid = threadIdx.x;
  if (tid < 64) hist[tid] = 0;
  double acc = 0.0;
  for (int i = tid; i < k; i += 256) acc += s[i] * s[i];
  red[tid] = acc;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) red[tid] += red[tid + h];
    __syncthreads();
  }
  const double tot = red[0];
  for (int i = tid; i < k; i += 256) {
    const double v = s[i] * s[i];
    int b = 0;
    if (v > 0.0 && tot > 0.0) {
      const double x = log10(v / tot);
      const double fb = floor((x + 16.0) / 0.25);
      b = fb < 0.0 ? 0 : (fb > 63.0 ? 63 : (int)fb);
    }
    atomicAdd(&hist[b], 1);
  }
  __syncthreads();
  if (tid < 64) feat[tid] = k > 0 ? (float)((double)hist[tid] / (double)k) : 0.0f;
  if (tid == 64) feat[64] = (float)bond_f;
  if (tid == 65) feat[65] = (float)cycle_f;
}

void spectrum_features(const double* s_dev, int k, int bond, int n_sites, int cycle, int n_cycles,
                       float* feat_dev, hipStream_t st) {
  const double bf = (double)bond / (double)std::max(n_sites - 2, 1);
  const double cf = (double)cycle / (double)std::max(n_cycles, 1);
  hipLaunchKernelGGL(k_spec_features, dim3(1), dim3(256), 0, st, s_dev, k, bf, cf, feat_dev);
  HIP_LAUNCH_OK();
}

// Training targets (32): y_j = log10(max(tail(ceil(m j/32)) / w, 1e-20)),
// j = 1..32, tail(k) = sum_{r>=k} s_r^2 accumulated from the smallest upward
// with values s^2 <= 1e-24 w counted as zero, w = sum s^2.
__global__ void k_spec_targets(const double* s, int m, float* y) {
  if (threadIdx.x != 0) return;
  double w = 0.0;
  for (int i = m - 1; i >= 0; --i) w += s[i] * s[i];
  const double floor_ = 1e-24 * w;
  double tail = 0.0;
  int next = NO;   // fill targets from j = 32 downward while walking k down
  for (int kk = m; kk >= 0; --kk) {
    // tail == tail(kk)
    while (next >= 1) {
      int kj = (int)ceil((double)next / NO * m);
      if (kj > m) kj = m;
      if (kj != kk) break;
      const double v = w > 0.0 ? tail / w : 0.0;
      y[next - 1] = (float)log10(fmax(v, 1e-20));
      --next;
    }
    if (kk == 0) break;
    const double v2 = s[kk - 1] * s[kk - 1];
    tail += v2 <= floor_ ? 0.0 : v2;
  }
}

void spectrum_targets(const double* s_dev, int m, float* y_dev, hipStream_t st) {
  hipLaunchKernelGGL(k_spec_targets, dim3(1), dim3(64), 0, st, s_dev, m, y_dev);
  HIP_LAUNCH_OK();
}

// ------------------------------------------------- forward and backward
// Two samples per block of 128 threads (thread t owns unit t of each layer),
// so that every weight read from L2 serves two samples; weight rows are read
// as vectors, activations stay in LDS (13 us at batch 256; the weights staged
// in LDS first: 14).  With `act` set (training) the block
// goes on to the deltas
//   dout = 2 (out - y) / (batch * 32), dz2 = (dout W3) . [h2 > 0],
//   dz1 = (dz2 W2) . [h1 > 0],
// stores h1, h2 ([batch][2][128]) and dz1, dz2, dout ([batch][288]) for the
// weight gradients, and each sample's sum of squared errors.
constexpr int MS = 2;                      // samples per block
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));   // the caller's arrays are only float-aligned
constexpr int DL = 2 * NH + NO;            // deltas per sample
__global__ __launch_bounds__(128) void k_mlp(const float* w, const float* x, const float* y, int batch, float* out,
                                             float* act, float* dl, float* sq) {
  __shared__ float xs[MS][NI + 2], h1[MS][NH], h2[MS][NH], dout[MS][NO], dz2[MS][NH];
  const int b0 = blockIdx.x * MS, t = threadIdx.x, ns = min(MS, batch - b0);
  for (int e = t; e < MS * NI; e += 128)
    xs[e / NI][e % NI] = e / NI < ns ? x[(int64_t)b0 * NI + e] : 0.f;
  __syncthreads();
  float z[MS];
  {
#pragma unroll
    for (int m = 0; m < MS; ++m) z[m] = w[OFF_B1 + t];
    const f2u* wr = reinterpret_cast<const f2u*>(w + OFF_W1 + t * NI);
#pragma unroll 11
    for (int i = 0; i < NI / 2; ++i) {
      const f2u v = wr[i];
#pragma unroll
      for (int m = 0; m < MS; ++m) z[m] = fmaf(v.y, xs[m][2 * i + 1], fmaf(v.x, xs[m][2 * i], z[m]));
    }
#pragma unroll
    for (int m = 0; m < MS; ++m) h1[m][t] = z[m] > 0.f ? z[m] : 0.f;
  }
  __syncthreads();
  {
#pragma unroll
    for (int m = 0; m < MS; ++m) z[m] = w[OFF_B2 + t];
    const f2u* wr = reinterpret_cast<const f2u*>(w + OFF_W2 + t * NH);
#pragma unroll 16
    for (int i = 0; i < NH / 2; ++i) {
      const f2u v = wr[i];
#pragma unroll
      for (int m = 0; m < MS; ++m) z[m] = fmaf(v.y, h1[m][2 * i + 1], fmaf(v.x, h1[m][2 * i], z[m]));
    }
#pragma unroll
    for (int m = 0; m < MS; ++m) h2[m][t] = z[m] > 0.f ? z[m] : 0.f;
  }
  __syncthreads();
  const int o = t % NO, m = t / NO;        // threads 0..63: output o of sample m
  if (m < ns) {
    float v = w[OFF_B3 + o];
    const f2u* wr = reinterpret_cast<const f2u*>(w + OFF_W3 + o * NH);
#pragma unroll 16
    for (int i = 0; i < NH / 2; ++i) v = fmaf(wr[i].y, h2[m][2 * i + 1], fmaf(wr[i].x, h2[m][2 * i], v));
    if (out) out[(int64_t)(b0 + m) * NO + o] = v;
    if (act) {
      const float d = v - y[(int64_t)(b0 + m) * NO + o];
      dout[m][o] = 2.0f / ((float)batch * (float)NO) * d;
      float q = d * d;
#pragma unroll
      for (int h = NO / 2; h > 0; h >>= 1) q += __shfl_xor(q, h);
      if (o == 0) sq[b0 + m] = q;
    }
  }
  if (!act) return;
  __syncthreads();
  {
    float d[MS];
#pragma unroll
    for (int k = 0; k < MS; ++k) d[k] = 0.f;
#pragma unroll 8
    for (int e = 0; e < NO; ++e) {
      const float v = w[OFF_W3 + e * NH + t];
#pragma unroll
      for (int k = 0; k < MS; ++k) d[k] = fmaf(dout[k][e], v, d[k]);
    }
#pragma unroll
    for (int k = 0; k < MS; ++k) dz2[k][t] = h2[k][t] > 0.f ? d[k] : 0.f;
  }
  __syncthreads();
  {
    float d[MS];
#pragma unroll
    for (int k = 0; k < MS; ++k) d[k] = 0.f;
#pragma unroll 16
    for (int e = 0; e < NH; ++e) {
      const float v = w[OFF_W2 + e * NH + t];
#pragma unroll
      for (int k = 0; k < MS; ++k) d[k] = fmaf(dz2[k][e], v, d[k]);
    }
    for (int k = 0; k < ns; ++k) {
      float* a = act + (int64_t)(b0 + k) * 2 * NH;
      float* g = dl + (int64_t)(b0 + k) * DL;
      a[t] = h1[k][t];
      a[NH + t] = h2[k][t];
      g[t] = h1[k][t] > 0.f ? d[k] : 0.f;
      g[NH + t] = dz2[k][t];
      if (t < NO) g[2 * NH + t] = dout[k][t];
    }
  }
}

// Weight gradients: a block takes a 16 x 16 tile of one weight matrix, its
// four waves a quarter of the batch each (two outputs by two inputs per
// lane), summed in wave order; the tiles of the first 16 inputs also sum the
// bias gradient.  The last block reduces the loss, mean (out - y)^2, over the
// samples' sums in a fixed tree.  (One thread per weight walking the whole
// batch took 65 us at batch 256.)
constexpr int GT = 16;
constexpr int TI1 = (NI + GT - 1) / GT, TI2 = NH / GT, TO = NH / GT, TO3 = NO / GT;
constexpr int WG_TILES = TO * TI1 + TO * TI2 + TO3 * TI2;
__global__ __launch_bounds__(256) void k_mlp_wgrad(const float* x, const float* act, const float* dl, const float* sq,
                                                   int batch, float* g, float* loss) {
  __shared__ float red[4][GT][GT + 1], rb[4][GT];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int tile = blockIdx.x;
  if (tile == WG_TILES) {
    if (!loss) return;
    float* r = &red[0][0][0];
    float acc = 0.f;
    for (int i = tid; i < batch; i += 256) acc += sq[i];
    r[tid] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) r[tid] += r[tid + h];
      __syncthreads();
    }
    if (tid == 0) *loss = r[0] / (float)(batch * NO);
    return;
  }
  const float *d, *a;
  int ni, lda, off_w, off_b, ti;
  if (tile < TO * TI1) {                    // W1: dz1, x
    d = dl;
    a = x;
    ni = NI;
    lda = NI;
    off_w = OFF_W1;
    off_b = OFF_B1;
    ti = TI1;
  } else if (tile < TO * TI1 + TO * TI2) {  // W2: dz2, h1
    tile -= TO * TI1;
    d = dl + NH;
    a = act;
    ni = NH;
    lda = 2 * NH;
    off_w = OFF_W2;
    off_b = OFF_B2;
    ti = TI2;
  } else {                                  // W3: dout, h2
    tile -= TO * TI1 + TO * TI2;
    d = dl + 2 * NH;
    a = act + NH;
    ni = NH;
    lda = 2 * NH;
    off_w = OFF_W3;
    off_b = OFF_B3;
    ti = TI2;
  }
  const int o0 = (tile / ti) * GT, i0 = (tile % ti) * GT;
  const int lo = 2 * (lane >> 3), li = 2 * (lane & 7);
  const bool in = i0 + li < ni;             // ni is even
  const f2u* dp = reinterpret_cast<const f2u*>(d + o0 + lo);
  const f2u* ap = reinterpret_cast<const f2u*>(a + i0 + (in ? li : 0));
  const int per = (batch + 3) / 4, b0 = w * per, b1 = min(batch, b0 + per);
  float s00 = 0.f, s01 = 0.f, s10 = 0.f, s11 = 0.f, t0 = 0.f, t1 = 0.f;
#pragma unroll 8
  for (int b = b0; b < b1; ++b) {
    const f2u dv = dp[(int64_t)b * (DL / 2)], av = ap[(int64_t)b * (lda / 2)];
    s00 = fmaf(dv.x, av.x, s00);
    s01 = fmaf(dv.x, av.y, s01);
    s10 = fmaf(dv.y, av.x, s10);
    s11 = fmaf(dv.y, av.y, s11);
    t0 += dv.x;
    t1 += dv.y;
  }
  red[w][lo][li] = s00;
  red[w][lo][li + 1] = s01;
  red[w][lo + 1][li] = s10;
  red[w][lo + 1][li + 1] = s11;
  if (li == 0) {
    rb[w][lo] = t0;
    rb[w][lo + 1] = t1;
  }
  __syncthreads();
  const int r = tid / GT, c = tid % GT;
  if (i0 + c < ni) g[off_w + (o0 + r) * ni + i0 + c] = ((red[0][r][c] + red[1][r][c]) + red[2][r][c]) + red[3][r][c];
  if (i0 == 0 && tid < GT) g[off_b + o0 + tid] = ((rb[0][tid] + rb[1][tid]) + rb[2][tid]) + rb[3][tid];
}

// Adam (Kingma & Ba 2015) with bias correction.
__global__ void k_adam(float* w, const float* g, float* m, float* v, int count, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

void mlp_forward(const float* w, const float* x, int batch, float* out, hipStream_t s) {
  if (batch <= 0) return;
  hipLaunchKernelGGL(k_mlp, dim3(ceil_div(batch, MS)), dim3(128), 0, s, w, x, nullptr, batch, out, nullptr, nullptr,
                     nullptr);
  HIP_LAUNCH_OK();
}

}  // namespace rcs

extern "C" {

#define RCS_API_BEGIN try {
#define RCS_API_END                  \
  }                                  \
  catch (const rcs::Error& e) {      \
    rcs::set_last_error(e.what());   \
    return e.status;                 \
  }                                  \
  catch (const std::exception& e) {  \
    rcs::set_last_error(e.what());   \
    return RCS_ERR_DEVICE;           \
  }                                  \
  return RCS_OK;

rcs_status rcs_spectrum_features(const double* s_dev, int32_t k, int32_t bond, int32_t n_sites,
                                 int32_t cycle, int32_t n_cycles, float* feat_dev, void* stream) {
  RCS_API_BEGIN
  RCS_REQUIRE(feat_dev && (s_dev || k == 0) && k >= 0, "bad arguments");
  rcs::spectrum_features(s_dev, k, bond, n_sites, cycle, n_cycles, feat_dev, rcs::as_stream(stream));
  RCS_API_END
}

rcs_status rcs_spectrum_targets(const double* s_dev, int32_t m, float* y_dev, void* stream) {
  RCS_API_BEGIN
  RCS_REQUIRE(s_dev && y_dev && m >= 1, "bad arguments");
  rcs::spectrum_targets(s_dev, m, y_dev, rcs::as_stream(stream));
  RCS_API_END
}

rcs_status rcs_mlp_forward(const float* w_dev, const float* x_dev, int32_t batch, float* out_dev,
                           void* stream) {
  RCS_API_BEGIN
  RCS_REQUIRE(w_dev && x_dev && out_dev && batch >= 0, "bad arguments");
  rcs::mlp_forward(w_dev, x_dev, batch, out_dev, rcs::as_stream(stream));
  RCS_API_END
}

rcs_status rcs_mlp_backward(const float* w_dev, const float* x_dev, const float* y_dev, int32_t batch,
                            float* grad_dev, float* loss_dev, void* stream) {
  RCS_API_BEGIN
  RCS_REQUIRE(w_dev && x_dev && y_dev && grad_dev && batch >= 1, "bad arguments");
  hipStream_t s = rcs::as_stream(stream);
  rcs::DevBuf ws;
  ws.ensure((size_t)batch * (2 * rcs::NH + rcs::DL + 1) * sizeof(float));
  float* act = ws.as<float>();
  float* dl = act + (size_t)batch * 2 * rcs::NH;
  float* sq = dl + (size_t)batch * rcs::DL;
  hipLaunchKernelGGL(rcs::k_mlp, dim3(rcs::ceil_div(batch, rcs::MS)), dim3(128), 0, s, w_dev, x_dev, y_dev, batch,
                     nullptr, act, dl, sq);
  HIP_LAUNCH_OK();
  hipLaunchKernelGGL(rcs::k_mlp_wgrad, dim3(rcs::WG_TILES + 1), dim3(256), 0, s, x_dev, act, dl, sq, batch, grad_dev,
                     loss_dev);
  HIP_LAUNCH_OK();
  HIP_OK(hipStreamSynchronize(s));
  RCS_API_END
}

rcs_status rcs_mlp_adam(float* w_dev, const float* grad_dev, float* m_dev, float* v_dev, int32_t count,
                        int32_t step, float lr, float beta1, float beta2, float eps, void* stream) {
  RCS_API_BEGIN
  RCS_REQUIRE(w_dev && grad_dev && m_dev && v_dev && count >= 0 && step >= 1, "bad arguments");
  const float c1 = 1.f - std::pow(beta1, (float)step), c2 = 1.f - std::pow(beta2, (float)step);
  if (count > 0) {
    hipLaunchKernelGGL(rcs::k_adam, dim3(rcs::ceil_div(count, 256)), dim3(256), 0, rcs::as_stream(stream), w_dev,
                       grad_dev, m_dev, v_dev, count, lr, beta1, beta2, eps, c1, c2);
    HIP_LAUNCH_OK();
  }
  RCS_API_END
}

}  // extern "C"
