// The two-site matrix (products A_i^{s1} A_{i+1}^{s2} mixed with the gate) in
// reduced precision.
//
//  complex64 : operands rounded to fp32, v_mfma_f32_16x16x4f32, fp32 sums;
//  split-bf16: each fp32 operand x = hi + lo with hi = bf16(x), lo =
//              bf16(x - hi) (round to nearest even); every real product is
//              hi*hi' + hi*lo' + lo*hi' on v_mfma_f32_16x16x32_bf16 with fp32
//              accumulation (Henry, Tang, Heinecke, ARITH 2019), complex
//              products in the four-real-product form.
// Site tensors stay complex128 in HBM; operands are converted while staged
// into LDS, once per element.  As in the fp64 kernel a workgroup computes the
// four products of a 32 x 32 tile (a, c) as one 64 x 64 tile of the stacked
// operands, one product per wave, exchanges them through LDS and writes the
// mixed complex128 result, so the products never go to memory.
//
// MFMA layouts (lane l): f32 16x16x4: A[l%16][l/16], B[l/16][l%16];
// bf16 16x16x32: A[l%16][8(l/16)+j], B[8(l/16)+j][l%16], j = 0..7;
// both: D[4(l/16)+r][l%16].
#include <hip/hip_ext.h>

#include "build.h"
#include "common.h"

namespace rcs {

constexpr int CT_T = 32;      // tile side in a and c
constexpr int CT_K = 32;      // k-values per stage
constexpr int CT_THREADS = 256;

// Staged operand rows x = (s, i) with k contiguous: fp32 planes (padded rows
// of 36), or bf16 planes (re hi, re lo, im hi, im lo) of 64-byte rows whose
// four 16-byte units are XOR-permuted by the row, so that the fragment reads
// (16 rows at one unit) and the writes spread over the banks.
struct StageF32 {
  float re[2 * CT_T][CT_K + 4], im[2 * CT_T][CT_K + 4];
};
struct StageBf16 {
  uint16_t v[4][2 * CT_T * CT_K];
};
__device__ inline int bf_off(int x, int k) { return x * CT_K + (((k >> 3) ^ ((x >> 2) & 3)) << 3) + (k & 7); }

__device__ inline uint16_t bf_bits(__bf16 h) {
  uint16_t b;
  __builtin_memcpy(&b, &h, 2);
  return b;
}
// The operand's fp32 value.  It must be rounded to fp32 before it is split:
// under contraction the compiler would merge both roundings into one from
// fp64 to bf16, which differs on double-rounding cases.
__device__ inline float fp32_value(double x) {
  float f = (float)x;
  asm("" : "+v"(f));
  return f;
}
// hi and lo parts of two neighbouring k-values, packed.
__device__ inline void split2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  const __bf16 h0 = (__bf16)x0, h1 = (__bf16)x1;
  const __bf16 l0 = (__bf16)(x0 - (float)h0), l1 = (__bf16)(x1 - (float)h1);
  hi = bf_bits(h0) | ((uint32_t)bf_bits(h1) << 16);
  lo = bf_bits(l0) | ((uint32_t)bf_bits(l1) << 16);
}
__device__ inline void put2(StageF32& s, int x, int k, const double2& v0, const double2& v1) {
  *reinterpret_cast<float2*>(&s.re[x][k]) = make_float2((float)v0.x, (float)v1.x);
  *reinterpret_cast<float2*>(&s.im[x][k]) = make_float2((float)v0.y, (float)v1.y);
}
__device__ inline void put2(StageBf16& s, int x, int k, const double2& v0, const double2& v1) {
  uint32_t hi, lo;
  const int o = bf_off(x, k);
  split2(fp32_value(v0.x), fp32_value(v1.x), hi, lo);
  *reinterpret_cast<uint32_t*>(&s.v[0][o]) = hi;
  *reinterpret_cast<uint32_t*>(&s.v[1][o]) = lo;
  split2(fp32_value(v0.y), fp32_value(v1.y), hi, lo);
  *reinterpret_cast<uint32_t*>(&s.v[2][o]) = hi;
  *reinterpret_cast<uint32_t*>(&s.v[3][o]) = lo;
}

struct AccLowp {
  float4_t re[2][2], im[2][2];
};

// One 32-deep stage: the wave's 32 x 32 product of rows wm.. and columns wn...
__device__ inline void mma_lowp(const StageF32& a, const StageF32& b, AccLowp& c, int wm, int wn, int lane) {
#pragma unroll
  for (int kk = 0; kk < CT_K; kk += 4) {
    const int k = kk + (lane >> 4);
    float ar[2], ai[2], br[2], bi[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      ar[t] = a.re[wm + t * 16 + (lane & 15)][k];
      ai[t] = a.im[wm + t * 16 + (lane & 15)][k];
      br[t] = b.re[wn + t * 16 + (lane & 15)][k];
      bi[t] = b.im[wn + t * 16 + (lane & 15)][k];
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        c.re[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[mt], br[nt], c.re[mt][nt], 0, 0, 0);
        c.re[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(-ai[mt], bi[nt], c.re[mt][nt], 0, 0, 0);
        c.im[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar[mt], bi[nt], c.im[mt][nt], 0, 0, 0);
        c.im[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai[mt], br[nt], c.im[mt][nt], 0, 0, 0);
      }
  }
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ inline bf16x8_t bf_frag(const StageBf16& s, int plane, int x, int lane) {
  return *reinterpret_cast<const bf16x8_t*>(&s.v[plane][bf_off(x + (lane & 15), 8 * (lane >> 4))]);
}
__device__ inline bf16x8_t bf_neg(bf16x8_t v) {
  u32x4 b;
  __builtin_memcpy(&b, &v, 16);
  b ^= 0x80008000u;
  __builtin_memcpy(&v, &b, 16);
  return v;
}
__device__ inline void mma_lowp(const StageBf16& a, const StageBf16& b, AccLowp& c, int wm, int wn, int lane) {
  bf16x8_t bf[4][2];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int t = 0; t < 2; ++t) bf[p][t] = bf_frag(b, p, wn + t * 16, lane);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const bf16x8_t arh = bf_frag(a, 0, wm + mt * 16, lane), arl = bf_frag(a, 1, wm + mt * 16, lane);
    const bf16x8_t aih = bf_frag(a, 2, wm + mt * 16, lane), ail = bf_frag(a, 3, wm + mt * 16, lane);
    const bf16x8_t naih = bf_neg(aih), nail = bf_neg(ail);
    const bf16x8_t ar[6] = {arh, arh, arl, naih, naih, nail}, ai[6] = {arh, arh, arl, aih, aih, ail};
    constexpr int pr[6] = {0, 1, 0, 2, 3, 2}, pi[6] = {2, 3, 2, 0, 1, 0};
    // Re += Ar Br - Ai Bi, Im += Ar Bi + Ai Br, each as hi hi', hi lo', lo hi'
#pragma unroll
    for (int e = 0; e < 6; ++e)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        c.re[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[e], bf[pr[e]][nt], c.re[mt][nt], 0, 0, 0);
        c.im[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[e], bf[pi[e]][nt], c.im[mt][nt], 0, 0, 0);
      }
  }
}

// Tile of this workgroup.  Consecutive workgroups go to the eight dies in
// turn, each with an L2 of its own, so die d takes the d-th eighth of an
// order that walks strips of six tile columns row by row: its tiles form a
// patch that shares operand rows and columns.  The width matters where the
// operands are several times an L2: at bond 2048 in split bf16 four to eight
// columns take 1.31 ms, one 1.41 and twelve 1.35; up to bond 1024 anything
// from three on is within 3%.
__device__ inline void xcd_tile(int& tx, int& ty) {
  const int gx = gridDim.x, gy = gridDim.y, n = gx * gy, id = blockIdx.y * gx + blockIdx.x;
  const int d = id & 7, q = n / 8, r = n % 8, t = d * q + min(d, r) + (id >> 3);
  constexpr int W = 6;
  const int whole = gx / W * W * gy, w = t < whole ? W : gx % W, u = t < whole ? t % (W * gy) : t - whole;
  tx = (t < whole ? t / (W * gy) * W : gx / W * W) + u % w;
  ty = u / w;
}

// Bound: the bf16 form by LDS and conversion (fp64 operands split into four
// 16-bit planes per tile; the MFMAs take a sixth of the time), the fp32 form by
// the fp32 matrix cores.  Loads are two stages ahead, the LDS stage is
// double-buffered.  At bonds 700, 1001, 517 the call takes 99 us in split bf16;
// 113 with predicated loads one stage ahead, tiles in launch order and B
// written by 64 columns at a time (four-way bank conflicts); 344 with the
// split made per fragment by every wave, the products written to memory and
// mixed from there, and operands copied to the device layout first.
template <class Stage>
__global__ __launch_bounds__(CT_THREADS) void k_two_site_mix_lowp(SiteView A, SiteView B, Gate4 G, int dl, int dm,
                                                                 int dr, MixOut out) {
  __shared__ union {
    struct {
      Stage a, b;
    } st[2];
    float2 t[4][CT_T][CT_T + 1];
  } u;
  int tx, ty;
  xcd_tile(tx, ty);
  const int a0 = ty * CT_T, c0 = tx * CT_T;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = (w & 1) * 32, wn = (w >> 1) * 32;      // wave (s1, s2)
  // A: 16 lanes cover the 32 k-values of a row (two each), four passes of 16
  // rows; B: 16 lanes along c, two k-values each, four passes of 16 columns (a
  // wave's LDS writes then cover 16 columns x 4 pairs, which is all banks)
  const int ak = 2 * (tid & 15), ax = tid >> 4;
  const int bx = tid & 15, bk = 2 * (tid >> 4);
  double2 pa[2][4][2], pb[2][4][2];   // stages s + 1 and s + 2
  // Loads without a predicate (a predicated one waits for the last): rows and
  // columns past the end repeat the last one and their products are not
  // stored, k-values past the end are cleared.
  const double2* arow[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int x = ax + 16 * j;
    arow[j] = A.p + (x >> 5) * A.s + (int64_t)min(a0 + (x & 31), dl - 1) * A.ld;
  }
  const double2* bcol[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int x = bx + 16 * j;
    bcol[j] = B.p + (x >> 5) * B.s + min(c0 + (x & 31), dr - 1);
  }
  auto fetch = [&](double2 (&ra)[4][2], double2 (&rb)[4][2], int k0) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) ra[j][h] = arow[j][min(k0 + ak + h, dm - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) rb[j][h] = bcol[j][(int64_t)min(k0 + bk + h, dm - 1) * B.ld];
    if (k0 + CT_K > dm) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (k0 + ak + h >= dm) ra[j][h] = make_double2(0.0, 0.0);
          if (k0 + bk + h >= dm) rb[j][h] = make_double2(0.0, 0.0);
        }
    }
  };
  auto commit = [&](const double2 (&ra)[4][2], const double2 (&rb)[4][2], int buf) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      put2(u.st[buf].a, ax + 16 * j, ak, ra[j][0], ra[j][1]);
      put2(u.st[buf].b, bx + 16 * j, bk, rb[j][0], rb[j][1]);
    }
  };
  AccLowp acc;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc.re[i][j] = float4_t{0, 0, 0, 0};
      acc.im[i][j] = float4_t{0, 0, 0, 0};
    }
  fetch(pa[0], pb[0], 0);
  if (CT_K < dm) fetch(pa[1], pb[1], CT_K);
  commit(pa[0], pb[0], 0);
  __syncthreads();
  for (int k0 = 0; k0 < dm; k0 += 2 * CT_K) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = k0 + h * CT_K;
      if (k >= dm) break;
      if (k + 2 * CT_K < dm) fetch(pa[h], pb[h], k + 2 * CT_K);
      mma_lowp(u.st[h].a, u.st[h].b, acc, wm, wn, lane);
      if (k + CT_K < dm) {
        commit(pa[h ^ 1], pb[h ^ 1], h ^ 1);
        __syncthreads();
      }
    }
  }
  __syncthreads();
  const int q = 2 * (w & 1) + (w >> 1);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        u.t[q][mt * 16 + 4 * (lane >> 4) + r][nt * 16 + (lane & 15)] =
            make_float2(acc.re[mt][nt][r], acc.im[mt][nt][r]);
  __syncthreads();
  for (int e = tid; e < CT_T * CT_T; e += CT_THREADS) {
    const int i = out.orient == 1 ? e % CT_T : e / CT_T, j = out.orient == 1 ? e / CT_T : e % CT_T;
    if (a0 + i < dl && c0 + j < dr) {
      double2 t[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) t[p] = make_double2(u.t[p][i][j].x, u.t[p][i][j].y);
      mix_store(t, G, a0 + i, c0 + j, dl, dr, out);
    }
  }
}

void contract_mix_lowp(const SiteView& A, const SiteView& B, const Gate4& G, int dl, int dm, int dr, int precision,
                       const MixOut& out, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(ceil_div(dr, CT_T), ceil_div(dl, CT_T));
  if (precision == RCS_PREC_C64)
    hipExtLaunchKernelGGL((k_two_site_mix_lowp<StageF32>), grid, dim3(CT_THREADS), 0, s, start, stop, 0, A, B, G, dl,
                          dm, dr, out);
  else
    hipExtLaunchKernelGGL((k_two_site_mix_lowp<StageBf16>), grid, dim3(CT_THREADS), 0, s, start, stop, 0, A, B, G, dl,
                          dm, dr, out);
  HIP_LAUNCH_OK();
}

}  // namespace rcs
