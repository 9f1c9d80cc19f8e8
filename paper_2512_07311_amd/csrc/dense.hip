// Dense state vector of the random circuit on one GPU, the exact reference
// for true-fidelity XEB (Section 5.1 scores samples against exact output
// probabilities).  psi has 2^n complex128 amplitudes, index i = sum_q b_q 2^q
// (bit q = qubit q, the bitstring convention); 34 qubits take 256 GiB.
//
// The vector goes through in passes.  A pass picks up to 12 qubits, always
// the 4 lowest among them (so that each global access moves 256 bytes); a
// workgroup stages the 2^12 amplitudes whose indices vary in those bits in
// LDS, applies every gate of the circuit that is next in line on qubits of
// the set, across layers and cycles, and writes the amplitudes back.
//
// A pass costs one read and write of psi (16 x 2^n bytes each way, the bound)
// and the gates' fp64 work, so passes are what is saved:
//  * the single-qubit gates between two couplers of a qubit are multiplied
//    into one 2x2 matrix and applied with the next coupler, in registers (one
//    LDS round trip for three gates); the matrix is a real rotation between
//    phases, and the phases are multiplied into the couplers on either side,
//    which leaves 52 instead of 88 fp64 operations per four amplitudes;
//  * the qubit set of a pass is the best of the contiguous windows and of a
//    set grown from the first gate in line, each step adding the qubits that
//    let most gates run per qubit added.
// 28 qubits (4 x 7), 8 cycles: 10 passes instead of the 64 that one window
// and one layer per pass took, 28.0 ms instead of 166 (2.7 ms per pass against
// 2.6: a pass now carries about 9 couplers with their gates; the copy rate
// alone would be 2.0).  With general 2x2 matrices and places worked out for
// every amplitude: 34.8 ms.
// Normwise error against extended precision, gate by gate in fp64 / here: 20
// qubits, 8 cycles 1.0e-15 / 0.8e-15; 12 qubits, 200 cycles 6.4e-15 / 3.0e-15
// (7.2e-15 with plain cosines and sines and the repeated rounding of the
// couplers left in).
#include <algorithm>
#include <array>
#include <vector>

#include "circuit.h"
#include "common.h"

namespace rcs {

constexpr int DW_TILE = 12;     // qubits per pass
constexpr int DW_LOW = 4;       // always-staged low bits
constexpr int DW_THREADS = 512;
constexpr int DW_MAXSTEPS = 24; // per launch: the steps travel as kernel arguments (4 KB)
constexpr int DW_SPAN = 8;      // couplers span fewer qubit numbers than this

// One step on tile bits ta, tb.
//  kCoupler, kCouplerUnit: real rotations [[c, -s], [s, c]] with m[0] = (ca, sa)
//    (times a factor) and m[1] = (cb, sb) on the two qubits, then the coupler with the phases
//    around it: m[2..7] = its entries 00, 11, 12, 21, 22, 33 (Unit: 00 is 1);
//  kGates2: 2x2 matrices m[0..3] and m[4..7]; kGate1: m[0..3] on ta only.
enum { kCoupler, kCouplerUnit, kGates2, kGate1 };
struct DenseStep {
  double2 m[8];
  int kind, ta, tb;
};

struct DensePass {
  int tbits, low;              // tile bits, of which the lowest `low` are qubits 0..low-1
  int bit[DW_TILE];            // qubit of each tile bit, ascending
  int nsteps, init;            // init: psi is |0...0> (not read)
  DenseStep st[DW_MAXSTEPS];
};
static_assert(sizeof(DensePass) + 64 <= 4096, "kernel argument space");

__global__ void k_dense_init(double2* psi, int64_t len) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (int64_t)gridDim.x * blockDim.x)
    psi[i] = make_double2(i == 0 ? 1.0 : 0.0, 0.0);
}

__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ inline double2 cfma(double2 a, double2 b, double2 c) {   // c + a b
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ inline void apply2(const double2* u, double2& x0, double2& x1) {
  const double2 y0 = cfma(u[1], x1, cmul(u[0], x0)), y1 = cfma(u[3], x1, cmul(u[2], x0));
  x0 = y0;
  x1 = y1;
}
__device__ inline void rotate2(double2 cs, double2& x0, double2& x1) {
  const double2 y0 = make_double2(fma(cs.x, x0.x, -cs.y * x1.x), fma(cs.x, x0.y, -cs.y * x1.y));
  x1 = make_double2(fma(cs.x, x1.x, cs.y * x0.x), fma(cs.x, x1.y, cs.y * x0.y));
  x0 = y0;
}

// LDS position of tile index t: bits 4 and 5 are folded into the low four, so
// that 16 consecutive work items stay conflict-free when a gate on one of the
// low bits (or on two neighbouring ones) makes them skip it.
__device__ inline int dw_pos(int t) { return t ^ (((t >> 4) & 1) * 15) ^ (((t >> 5) & 1) * 5); }
// t with a zero bit inserted at position b.
__device__ inline int dw_insert0(int t, int b) { return ((t >> b) << (b + 1)) | (t & ((1 << b) - 1)); }

// One workgroup per combination of the bits outside the tile.
__global__ __launch_bounds__(DW_THREADS) void k_dense_pass(double2* psi, DensePass P) {
  extern __shared__ double2 tile[];
  __shared__ int64_t hi[1 << (DW_TILE - DW_LOW)];
  const int tsz = 1 << P.tbits, lowmask = (1 << P.low) - 1;
  int64_t base = blockIdx.x;
  for (int k = 0; k < P.tbits; ++k) base = ((base >> P.bit[k]) << (P.bit[k] + 1)) | (base & ((int64_t(1) << P.bit[k]) - 1));
  for (int v = threadIdx.x; v < (tsz >> P.low); v += DW_THREADS) {
    int64_t h = 0;
    for (int k = P.low; k < P.tbits; ++k) h |= (int64_t)((v >> (k - P.low)) & 1) << P.bit[k];
    hi[v] = h;
  }
  __syncthreads();
  constexpr int PER = (1 << DW_TILE) / DW_THREADS;
  // a full tile takes the loops without the bound: a predicated load waits for
  // the one before it
  const bool full = P.tbits == DW_TILE && !P.init;
  double2 r[PER];
  if (full) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int t = threadIdx.x + j * DW_THREADS;
      r[j] = psi[base + (t & lowmask) + hi[t >> P.low]];
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) tile[dw_pos(threadIdx.x + j * DW_THREADS)] = r[j];
  } else {
    for (int t = threadIdx.x; t < tsz; t += DW_THREADS) {
      const int64_t i = base + (t & lowmask) + hi[t >> P.low];
      tile[dw_pos(t)] = P.init ? make_double2(i == 0 ? 1.0 : 0.0, 0.0) : psi[i];
    }
  }
  __syncthreads();
  for (int o = 0; o < P.nsteps; ++o) {
    const DenseStep& S = P.st[o];
    if (S.kind == kGate1) {
      for (int p = threadIdx.x; p < (tsz >> 1); p += DW_THREADS) {
        const int t0 = dw_pos(dw_insert0(p, S.ta)), t1 = dw_pos(dw_insert0(p, S.ta) | (1 << S.ta));
        double2 x0 = tile[t0], x1 = tile[t1];
        apply2(S.m, x0, x1);
        tile[t0] = x0;
        tile[t1] = x1;
      }
    } else {
      // dw_insert0 and dw_pos are linear over the bits of the index, so the
      // places of a thread's later items and of an item's other three
      // amplitudes are its first place XOR a number that is the same for all
      const int lo = min(S.ta, S.tb), hb = max(S.ta, S.tb);
      const int pa = dw_pos(1 << S.ta), pb = dw_pos(1 << S.tb);
      const int p0 = dw_pos(dw_insert0(dw_insert0(threadIdx.x, lo), hb));
      for (int p = 0; p + (int)threadIdx.x < (tsz >> 2); p += DW_THREADS) {
        const int t00 = p0 ^ dw_pos(dw_insert0(dw_insert0(p, lo), hb)), t01 = t00 ^ pb, t10 = t00 ^ pa,
                  t11 = t01 ^ pa;
        double2 x00 = tile[t00], x01 = tile[t01], x10 = tile[t10], x11 = tile[t11];
        if (S.kind == kGates2) {
          apply2(S.m, x00, x10);
          apply2(S.m, x01, x11);
          apply2(S.m + 4, x00, x01);
          apply2(S.m + 4, x10, x11);
        } else {
          rotate2(S.m[0], x00, x10);
          rotate2(S.m[0], x01, x11);
          rotate2(S.m[1], x00, x01);
          rotate2(S.m[1], x10, x11);
          const double2 y01 = cfma(S.m[4], x10, cmul(S.m[3], x01)), y10 = cfma(S.m[6], x10, cmul(S.m[5], x01));
          if (S.kind == kCoupler) x00 = cmul(S.m[2], x00);
          x01 = y01;
          x10 = y10;
          x11 = cmul(S.m[7], x11);
        }
        tile[t00] = x00;
        tile[t01] = x01;
        tile[t10] = x10;
        tile[t11] = x11;
      }
    }
    __syncthreads();
  }
  for (int j = 0; j < PER; ++j) {
    const int t = threadIdx.x + j * DW_THREADS;
    if (t < tsz) psi[base + (t & lowmask) + hi[t >> P.low]] = tile[dw_pos(t)];
  }
}

namespace {

// Gates are few and repeat, so a rounding error in one would add up over the
// circuit instead of averaging out: the matrices are prepared in extended
// precision.
using xcplx = std::complex<long double>;
using Mat2 = std::array<xcplx, 4>;
Mat2 mul(const Mat2& a, const Mat2& b) {
  return Mat2{a[0] * b[0] + a[1] * b[2], a[0] * b[1] + a[1] * b[3], a[2] * b[0] + a[3] * b[2],
              a[2] * b[1] + a[3] * b[3]};
}
const Mat2 kIdentity{xcplx(1.0L), xcplx(0.0L), xcplx(0.0L), xcplx(1.0L)};
Mat2 gate_matrix(int g) {
  const auto u = one_qubit_gate(g);
  return Mat2{xcplx(u[0]), xcplx(u[1]), xcplx(u[2]), xcplx(u[3])};
}

// A coupler with the single-qubit gates since the previous coupler of each of
// its qubits, as real rotations times a factor (c, s) and the entries 00, 11,
// 12, 21, 22, 33 of the coupler with phases.
struct Block {
  int a, b;
  double ca, sa, cb, sb;
  xcplx f[6];
};

// A unitary u = common diag(1, d1) [[c, -s], [s, c]] diag(1, d2), the larger of
// c and s being 1: each of the gates on its own is a turn by a right angle, c =
// s = 1, which multiplies exactly.  common also holds what the other one lost
// in rounding.
struct Euler {
  xcplx common, d1, d2;
  double c, s;
};
Euler euler(const Mat2& u) {
  auto unit = [](const xcplx& z) { return std::abs(z) > 0.0L ? z / std::abs(z) : xcplx(1.0L); };
  const long double c = std::abs(u[0]), s = std::abs(u[2]);
  const xcplx p0 = unit(u[0]), p1 = unit(u[2]);
  Euler e;
  const long double m = std::max(c, s);
  e.c = (double)(c / m);
  e.s = (double)(s / m);
  e.d1 = p1 / p0;
  // the larger of cos and sin gives the second phase: u11 = p1 c d2, u01 = -p0 s d2
  e.d2 = c >= s ? unit(u[3]) / p1 : -unit(u[1]) / p0;
  e.common = p0 * (std::hypot(c, s) / std::hypot((long double)e.c, (long double)e.s));
  return e;
}

// The circuit as blocks per qubit, in order, and what is left to run.
struct Planner {
  int n;
  std::vector<Block> blocks;
  std::vector<std::vector<int>> line;   // blocks of each qubit
  std::vector<Mat2> last;               // gates after a qubit's last block
  std::vector<char> last_left;
  std::vector<int> next;                // position in line

  // Runs what a set of qubits allows from the positions nx, at most
  // DW_MAXSTEPS steps.  Returns a score (two per block, one per last gate);
  // `ran` (nullable) receives the blocks in order.
  int run(uint64_t set, std::vector<int>& nx, std::vector<int>* ran) const {
    int steps = 0;
    bool again = true;
    while (again && steps < DW_MAXSTEPS) {
      again = false;
      for (uint64_t m = set; m && steps < DW_MAXSTEPS; m &= m - 1) {
        const int q = __builtin_ctzll(m);
        while (nx[q] < (int)line[q].size() && steps < DW_MAXSTEPS) {
          const int i = line[q][nx[q]];
          const int o = blocks[i].a == q ? blocks[i].b : blocks[i].a;
          if (!((set >> o) & 1) || line[o][nx[o]] != i) break;
          ++nx[q];
          ++nx[o];
          ++steps;
          again = true;
          if (ran) ran->push_back(i);
        }
      }
    }
    int score = 2 * steps, lasts = 0;
    for (uint64_t m = set; m; m &= m - 1) {
      const int q = __builtin_ctzll(m);
      lasts += last_left[q] && nx[q] == (int)line[q].size();
    }
    return score + std::min(lasts, 2 * (DW_MAXSTEPS - steps));
  }

  // Set grown from a seed: adds, as long as qubits fit, the one or two that
  // raise the score most per qubit.
  uint64_t grow(uint64_t set, int room) const {
    std::vector<int> nx, ny;
    while (room > 0) {
      nx = next;
      const int s0 = run(set, nx, nullptr);
      uint64_t best = 0;
      double gain = 0.0;
      auto offer = [&](uint64_t add) {
        const int k = __builtin_popcountll(add);
        if (k == 0 || k > room) return;
        ny = next;
        const double g = (double)(run(set | add, ny, nullptr) - s0) / k;
        if (g > gain) {
          gain = g;
          best = add;
        }
      };
      for (int q = 0; q < n; ++q) {
        if (nx[q] < (int)line[q].size()) {
          const Block& b = blocks[line[q][nx[q]]];
          if (q == b.a || !((set >> b.a) & 1)) offer(((uint64_t(1) << b.a) | (uint64_t(1) << b.b)) & ~set);
        } else if (last_left[q] && !((set >> q) & 1)) {
          offer(uint64_t(1) << q);
        }
      }
      if (!best) break;
      set |= best;
      room -= __builtin_popcountll(best);
    }
    return set;
  }

  bool done() const {
    for (int q = 0; q < n; ++q)
      if (next[q] < (int)line[q].size() || last_left[q]) return false;
    return true;
  }
};

// Rows and columns (2 a + b) of a coupler's entries.
constexpr int kCouplerRow[6] = {0, 1, 1, 2, 2, 3}, kCouplerCol[6] = {0, 1, 2, 1, 2, 3};

void to_dev(const Mat2& m, double2* d) {
  for (int e = 0; e < 4; ++e) d[e] = make_double2((double)m[e].real(), (double)m[e].imag());
}

}  // namespace

void dense_simulate(const rcs_circuit_s& c, double2* psi, hipStream_t s) {
  const int n = c.n;
  for (int t = 0; t < c.n_cycles; ++t)
    for (auto& e : c.layers_2q[t])
      RCS_REQUIRE(std::abs(e.first - e.second) < std::min(DW_SPAN, n), "coupler wider than the dense window");
  Planner pl;
  pl.n = n;
  pl.line.resize(n);
  pl.next.assign(n, 0);
  pl.last.assign(n, kIdentity);
  pl.last_left.assign(n, 0);
  auto layer_1q = [&](const std::vector<int>& g) {
    for (int q = 0; q < n; ++q) {
      pl.last[q] = mul(gate_matrix(g[q]), pl.last[q]);
      pl.last_left[q] = 1;
    }
  };
  // Factors common to all amplitudes, collected per qubit line until they are
  // worth a multiply of a coupler's entry 00.  Whatever order the passes run
  // the couplers in, amplitudes are then too large by no more than what is on
  // its way along the lines, 2^16 for each of at most 36.  (Collected over the
  // circuit instead, the factors can all land on couplers that do not touch
  // some qubits, whose own couplers may run first, hundreds in a row.)
  std::vector<xcplx> owed(n, xcplx(1.0L));
  for (int t = 0; t < c.n_cycles; ++t) {
    layer_1q(c.layers_1q[t]);
    for (auto& e : c.layers_2q[t]) {
      const int a = std::min(e.first, e.second), b = std::max(e.first, e.second);
      // The rotations' inner phases go to the coupler, their outer ones to the
      // qubit's previous coupler (a phase of one qubit commutes with all that
      // acts on others; on |0> it is nothing), their common one to the first.
      const Euler ea = euler(pl.last[a]), eb = euler(pl.last[b]);
      Block B{a, b, ea.c, ea.s, eb.c, eb.s, {}};
      for (int e = 0; e < 6; ++e) {
        const int row = kCouplerRow[e], col = kCouplerCol[e];
        B.f[e] = xcplx(c.fsim[4 * row + col]) * (col & 2 ? ea.d1 : xcplx(1.0L)) * (col & 1 ? eb.d1 : xcplx(1.0L));
      }
      owed[a] *= owed[b] * ea.common * eb.common;
      owed[b] = xcplx(1.0L);
      if (std::abs(owed[a]) < 0x1p-16L) {
        for (xcplx& f : B.f) f *= owed[a];
        owed[a] = xcplx(1.0L);
      }
      for (int q : {a, b}) {
        if (!pl.line[q].empty()) {
          Block& prev = pl.blocks[pl.line[q].back()];
          for (int e = 0; e < 6; ++e)
            if (kCouplerRow[e] & (q == prev.a ? 2 : 1)) prev.f[e] *= q == a ? ea.d2 : eb.d2;
        }
        pl.line[q].push_back((int)pl.blocks.size());
      }
      pl.blocks.push_back(B);
      for (int q : {a, b}) {
        pl.last[q] = kIdentity;
        pl.last_left[q] = 0;
      }
    }
  }
  // The first coupler takes the rest, and the mean of what rounding to fp64 does
  // to the others: a gate that repeats repeats its error, which would otherwise
  // grow with the number of couplers instead of its root.
  xcplx common(1.0L);
  for (const xcplx& f : owed) common *= f;
  for (size_t i = 1; i < pl.blocks.size(); ++i) {
    xcplx num(0.0L);
    long double den = 0.0L;
    for (const xcplx& f : pl.blocks[i].f) {
      num += xcplx((double)f.real(), (double)f.imag()) * std::conj(f);
      den += std::norm(f);
    }
    common *= den / num;
  }
  if (!pl.blocks.empty())
    for (xcplx& f : pl.blocks[0].f) f *= common;
  if (c.final_layer && c.layers_1q.size() > (size_t)c.n_cycles) layer_1q(c.layers_1q[c.n_cycles]);

  const int low = std::min(DW_LOW, n), tbits = std::min(DW_TILE, n);
  const uint64_t lowset = (uint64_t(1) << low) - 1;
  DensePass P{};
  P.init = 1;
  if (pl.done()) {   // no gate at all
    const int64_t len = int64_t(1) << n;
    hipLaunchKernelGGL(k_dense_init, dim3((unsigned)std::min<int64_t>((len + 255) / 256, 1 << 20)), dim3(256), 0, s,
                       psi, len);
    HIP_LAUNCH_OK();
    return;
  }
  const int64_t groups = int64_t(1) << (n - tbits);
  RCS_REQUIRE(groups <= (int64_t(1) << 31) - 1, "state vector too large for the grid");
  std::vector<int> nx, ran;
  while (!pl.done()) {
    // the qubit set
    uint64_t set = (uint64_t(1) << n) - 1;
    if (n > tbits) {
      int best = -1;
      auto offer = [&](uint64_t cand) {
        nx = pl.next;
        const int sc = pl.run(cand, nx, nullptr);
        if (sc > best) {
          best = sc;
          set = cand;
        }
      };
      uint64_t seed = 0;
      for (int i = 0; i < (int)pl.blocks.size() && !seed; ++i) {
        const Block& b = pl.blocks[i];
        if (pl.next[b.a] < (int)pl.line[b.a].size() && pl.line[b.a][pl.next[b.a]] == i)
          seed = (uint64_t(1) << b.a) | (uint64_t(1) << b.b);
      }
      offer(pl.grow(lowset | seed, tbits - __builtin_popcountll(lowset | seed)));
      for (int w = low; w + (tbits - low) <= n; ++w) offer(lowset | (((uint64_t(1) << (tbits - low)) - 1) << w));
      // exactly tbits qubits: fill up with the lowest ones left
      for (int q = 0; q < n && __builtin_popcountll(set) < tbits; ++q) set |= uint64_t(1) << q;
    }
    P.tbits = tbits;
    P.low = low;
    int pos[64], k = 0;
    for (uint64_t m = set; m; m &= m - 1) {
      const int q = __builtin_ctzll(m);
      pos[q] = k;
      P.bit[k++] = q;
    }
    // its steps
    ran.clear();
    pl.run(set, pl.next, &ran);
    P.nsteps = 0;
    for (int i : ran) {
      DenseStep& S = P.st[P.nsteps++];
      const Block& B = pl.blocks[i];
      S.kind = B.f[0] == xcplx(1.0L) ? kCouplerUnit : kCoupler;
      S.ta = pos[B.a];
      S.tb = pos[B.b];
      S.m[0] = make_double2(B.ca, B.sa);
      S.m[1] = make_double2(B.cb, B.sb);
      for (int e = 0; e < 6; ++e) S.m[2 + e] = make_double2((double)B.f[e].real(), (double)B.f[e].imag());
    }
    int held = -1;   // a last gate waiting for a partner
    for (uint64_t m = set; m; m &= m - 1) {
      const int q = __builtin_ctzll(m);
      if (!pl.last_left[q] || pl.next[q] < (int)pl.line[q].size()) continue;
      if (held >= 0) {
        DenseStep& S = P.st[P.nsteps - 1];
        S.kind = kGates2;
        S.tb = pos[q];
        to_dev(pl.last[q], S.m + 4);
        held = -1;
      } else {
        if (P.nsteps == DW_MAXSTEPS) break;
        DenseStep& S = P.st[P.nsteps++];
        S.kind = kGate1;
        S.ta = pos[q];
        S.tb = 0;
        to_dev(pl.last[q], S.m);
        held = q;
      }
      pl.last_left[q] = 0;
    }
    hipLaunchKernelGGL(k_dense_pass, dim3((unsigned)groups), dim3(DW_THREADS), (size_t(1) << tbits) * sizeof(double2), s,
                       psi, P);
    HIP_LAUNCH_OK();
    P.init = 0;
  }
}

// out[i] = psi[bits[i]] (mode 0: amplitude, complex) or |psi[bits[i]]|^2
// (mode 1: probability, real).
__global__ void k_dense_gather(const double2* psi, int n, const uint64_t* bits, uint64_t m, int mode, void* out) {
  const uint64_t mask = n == 64 ? ~0ull : ((1ull << n) - 1);
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
    const double2 a = psi[bits[i] & mask];
    if (mode == 0)
      static_cast<double2*>(out)[i] = a;
    else
      static_cast<double*>(out)[i] = a.x * a.x + a.y * a.y;
  }
}

void dense_gather(const double2* psi, int n, const uint64_t* bits, uint64_t m, int mode, void* out, hipStream_t s) {
  if (m == 0) return;
  hipLaunchKernelGGL(k_dense_gather, dim3((unsigned)std::min<uint64_t>((m + 255) / 256, 65535)), dim3(256), 0, s, psi,
                     n, bits, m, mode, out);
  HIP_LAUNCH_OK();
}

}  // namespace rcs

extern "C" {

rcs_status rcs_dense_simulate(rcs_circuit c, double* psi_dev, int64_t n_amps, void* stream) {
  try {
    RCS_REQUIRE(c && psi_dev, "null argument");
    RCS_REQUIRE(c->n <= 36, "dense state vector limited to 36 qubits");
    RCS_REQUIRE(n_amps == (int64_t(1) << c->n), "psi must hold exactly 2^n amplitudes");
    rcs::dense_simulate(*c, reinterpret_cast<double2*>(psi_dev), rcs::as_stream(stream));
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

rcs_status rcs_dense_gather(const double* psi_dev, int32_t n_qubits, const uint64_t* bits_dev, uint64_t m,
                            int32_t probabilities, double* out_dev, void* stream) {
  try {
    RCS_REQUIRE(psi_dev && (bits_dev || m == 0) && (out_dev || m == 0), "null device pointer");
    RCS_REQUIRE(n_qubits >= 1 && n_qubits <= 36, "n_qubits out of range");
    rcs::dense_gather(reinterpret_cast<const double2*>(psi_dev), n_qubits, bits_dev, m, probabilities ? 1 : 0,
                      out_dev, rcs::as_stream(stream));
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

}  // extern "C"
