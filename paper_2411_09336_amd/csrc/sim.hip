// Batched truncated MPS simulation of the feature-map circuit (Sec. II-B,
// Fig. 1; circuit of Sec. II-C).
//
// Every circuit of a batch shares one gate list, hence one step list (runs
// of Rz records, centre moves and two-qubit gates); a launch runs a chunk of
// steps with one workgroup per circuit, each walking its own circuit through
// the chunk.  Rz layers are diagonal and applied in place (Fig. 1a).  A
// two-qubit gate on sites (p, p+1) (Fig. 1b):
//   * theta[(s,a),(t,b)] = sum_{s',t'} G[st,s't'] P[(s',a),(t',b)] with the
//     pair product P[(s',a),(t',b)] = sum_c A_p[s'][a][c] A_{p+1}[t'][c][b],
//     formed once per step as a block-wide GEMM through LDS;
//   * its SVD is taken by one-sided (Hestenes) Jacobi in FP64: pairs of
//     columns are rotated until every pair is orthogonal to relative
//     tolerance 1e-14; the columns then are U S.  To absorb S to the right
//     the columns of theta are orthogonalised (U = W / |W|, the new right
//     tensor is U^H theta); to absorb it to the left the columns of theta^H
//     are (giving V, the new left tensor is theta V).  The isometric factor
//     is therefore always a set of normalised Jacobi columns and the other
//     factor an exact projection, so no V matrix is accumulated;
//   * truncation keeps k = max(1, min(chi, k_cut)) columns by decreasing norm
//     (Eq. (8): k_cut is the smallest count whose discarded weight is at most
//     cutoff times the total; cutoff <= 0 keeps all non-zero columns) and the
//     kept weight is renormalised to one.
// Orthogonality-centre moves (canonicalisation before each truncation) use
// the same machinery without truncation: the site matrix is orthogonalised
// and the remainder is pushed into the neighbour via the identity two-site
// theta.
//
// Register layout of the Jacobi matrix M (<= 128 x 128 complex): the lanes of
// a wave are column pairs (positions 2 cp and 2 cp + 1, slots A and B) times
// row groups, and the waves share the rows.  Rounds alternate between pairs
// inside a lane and pairs across neighbouring lanes (odd-even transposition
// ordering, each pair exchanged after its rotation), so n rounds visit every
// pair once per sweep and the only data movement is one DPP lane shift each
// way in every second round.  Each round the partial inner products of the
// waves go through LDS.  Up to 64 x 64 every wave adds them up and forms the
// rotations of its own lanes; at 128 four waves form them for all.  A matrix
// up to 16 x 16 lies in one wave, which needs neither LDS nor barriers for its
// rounds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "qk_internal.h"

namespace qk {

namespace {

constexpr int kSvWaves = 16;              // waves of the wide step
constexpr int kSvThreads = kSvWaves * 64; // 1024
constexpr int kSvMaxN = 128;
constexpr int kMaxSweeps = 30;
// Two-site steps next to a bond above 64 (bond caps up to 128): Jacobi
// matrices up to 256 x 256 in a per-circuit slot of global scratch (two
// matrices of 1 MiB and 128 reflection vectors).
constexpr int kWideN = 256;
constexpr int kWideFrom = 64;     // a neighbouring bond above this takes the wide step
constexpr size_t kWideSlot = size_t(2) * kWideN * kWideN + kSvMaxN * kWideN + kSvMaxN;
constexpr double kJacobiTol = 1e-14;
// A sweep whose rotations all have |<X,Y>| below kJacobiLarge |X| |Y| ends
// the iteration: cyclic Jacobi converges quadratically, so the next sweep's
// would fall below kJacobiTol and rotate nothing.
constexpr double kJacobiLarge = 1e-8;
// columns whose weight is below this fraction of ||M||_F^2 are numerical zeros
constexpr double kZeroWeight = 1e-28;
constexpr double kDegenerateGap = 1e-10;

enum SvMode { GATE_RIGHT = 0, GATE_LEFT = 1, MOVE_RIGHT = 2, MOVE_LEFT = 3 };
enum GateOp { OP_RZ = 0, OP_RXX = 1, OP_SWAP = 2, OP_ID = 3 };

struct SvParams {
  double2 *f64;
  int64_t mps_stride;
  const int64_t *site_off;
  const int32_t *pad;
  int32_t *dims;
  int32_t m;
  int32_t chi;
  int32_t gate_split;  // cap the kept count at rank(G) x the middle bond
  double coef_xx;
  double cutoff;
  const double *X;
  int64_t ldx;
  double2 *scratch;  // per circuit: pair product (matrices above 32 x 32)
  int64_t scratch_stride;
  double2 *wscratch; // per circuit kWideSlot (bond caps above 64), else nullptr
  double *disc;
  double *maxdisc;
  int32_t *degen;
  int32_t *unconv;
  int64_t n;
  int32_t *trace;     // optional: per circuit and two-qubit gate (cut bond, sum_l D_l D_{l+1})
  int32_t trace_n2q;  // two-qubit gates per circuit (row length of the trace / 2)
  const int64_t *base;  // graph replays: first circuit of the replay (nullptr: 0)
};

// Circuit of this workgroup: workgroup i of a launch simulates circuit
// base + i, where base is read from device memory in a graph replay (each
// replay advances it by the launch's grid) and is 0 otherwise.  The SVD
// scratch slot is the workgroup index, so a graph needs scratch only for
// the circuits of one replay.
__device__ inline int64_t circuit_of(const int64_t *base) { return (base ? *base : 0) + blockIdx.x; }

// DPP lane moves of a double.  Lanes without a source lane receive zero
// (bound_ctrl), so no copy of the source is needed as the fallback value.
template <int CTRL>
__device__ inline double dpp_mov(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  return __hiloint2double(__builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, true));
}
// shr1: lane l receives lane l-1 (lane 0: zero); shl1: lane l receives lane
// l+1 (lane 63: zero)
__device__ inline double dpp_shr1(double x) { return dpp_mov<0x138>(x); }
__device__ inline double dpp_shl1(double x) { return dpp_mov<0x130>(x); }

// Sum over the 16 lanes of a DPP row (all 16 lanes receive the total).
__device__ inline double row_sum16(double x) {
  x += dpp_mov<0x128>(x);   // row_ror:8
  x += dpp_mov<0x124>(x);   // row_ror:4
  x += dpp_mov<0x122>(x);   // row_ror:2
  x += dpp_mov<0x121>(x);   // row_ror:1
  return x;
}

__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

// Lane-half and row exchanges of two doubles (gfx950 permlane swaps):
// swap32 leaves a = [a_lo, b_lo], b = [a_hi, b_hi] (32-lane halves);
// swap16 leaves a = [a_0, b_0, a_2, b_2], b = [a_1, b_1, a_3, b_3] (rows).
__device__ inline void swap32(double &a, double &b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  a = __hiloint2double(int(hi[0]), int(lo[0]));
  b = __hiloint2double(int(hi[1]), int(lo[1]));
}
__device__ inline void swap16(double &a, double &b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  a = __hiloint2double(int(hi[0]), int(lo[0]));
  b = __hiloint2double(int(hi[1]), int(lo[1]));
}

// Sum over the 64 lanes of the wave (every lane receives the total).
__device__ inline double wave_sum(double x) {
  x = row_sum16(x);
  double y = x;
  swap16(x, y);
  x += y;
  y = x;
  swap32(x, y);
  return x + y;
}

// 1 / x for x > 0 (hardware estimate and two Newton steps).
__device__ inline double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(r, fma(-x, r, 1.0), r);
  return fma(r, fma(-x, r, 1.0), r);
}

// Largest of the wave's unsigned values, in every lane.
__device__ inline uint32_t wave_max_bits(uint32_t v) {
  v = max(v, uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x128, 0xf, 0xf, true)));   // row_ror 8, 4, 2, 1
  v = max(v, uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x124, 0xf, 0xf, true)));
  v = max(v, uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x122, 0xf, 0xf, true)));
  v = max(v, uint32_t(__builtin_amdgcn_mov_dpp(int(v), 0x121, 0xf, 0xf, true)));
  auto a = __builtin_amdgcn_permlane16_swap(int(v), int(v), false, false);
  v = max(uint32_t(a[0]), uint32_t(a[1]));
  a = __builtin_amdgcn_permlane32_swap(int(v), int(v), false, false);
  return max(uint32_t(a[0]), uint32_t(a[1]));
}

// Sixteen wave sums at once (every lane receives all sixteen totals): a
// reduce-scatter over the lane halves and rows (each exchange halves the
// values a lane carries), a row sum of the remaining four, then the reverse
// exchanges to spread the totals.  About a third of the instructions of
// sixteen separate wave sums.
__device__ inline void wave_sum16(double (&v)[16]) {
  double u[8], t[4];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    swap32(v[2 * k], v[2 * k + 1]);
    u[k] = v[2 * k] + v[2 * k + 1];  // lanes 0-31: value 2k, lanes 32-63: value 2k+1
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    swap16(u[2 * k], u[2 * k + 1]);
    // rows 0, 1, 2, 3: values 4k, 4k+2, 4k+1, 4k+3, each over 4 lanes
    t[k] = row_sum16(u[2 * k] + u[2 * k + 1]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    double a = t[k], b = t[k];
    swap16(a, b);  // rows 0, 1: a = value 4k, b = 4k+2; rows 2, 3: a = 4k+1, b = 4k+3
    double a2 = a, b2 = b;
    swap32(a, a2);
    swap32(b, b2);
    v[4 * k] = a;
    v[4 * k + 1] = a2;
    v[4 * k + 2] = b;
    v[4 * k + 3] = b2;
  }
}

// Sixteen sums over the 32 lanes of each half, by one exchange between its
// rows: eight row sums instead of sixteen.
__device__ inline void half_sum16(double (&v)[16]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    swap16(v[2 * k], v[2 * k + 1]);
    double a = row_sum16(v[2 * k] + v[2 * k + 1]), b = a;   // rows 0, 2: value 2k, rows 1, 3: 2k + 1
    swap16(a, b);
    v[2 * k] = a;
    v[2 * k + 1] = b;
  }
}

// Four wave sums at once, as wave_sum16; identical in every lane.
__device__ inline void wave_sum4(double (&v)[4]) {
  swap32(v[0], v[1]);
  swap32(v[2], v[3]);
  double a = v[0] + v[1], b = v[2] + v[3];
  swap16(a, b);
  a = row_sum16(a + b);   // rows 0, 1, 2, 3: values 0, 2, 1, 3
  b = a;
  swap16(a, b);
  v[0] = v[1] = a;
  v[2] = v[3] = b;
  swap32(v[0], v[1]);
  swap32(v[2], v[3]);
}

// A value of lane 0, in every lane (wave-uniform control flow and
// identical rotation parameters across the rows of a column pair).
__device__ inline double lane0(double x) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                          __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// Values that are the same in every lane, moved to scalar registers: the
// steps are separate functions, whose arguments arrive in vector registers.
__device__ inline int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline int64_t uniform(int64_t x) {
  return int64_t((uint64_t(uint32_t(uniform(int(uint64_t(x) >> 32)))) << 32) | uint32_t(uniform(int(x))));
}
// A structure in device memory that no kernel writes, read by scalar loads.
template <typename S>
__device__ inline S uniform_load(const S *p) {
  typedef const S __attribute__((address_space(4))) * Const;
  S r;
  __builtin_memcpy(&r, (const S *)(Const)(uniform(reinterpret_cast<int64_t>(p))), sizeof(S));
  return r;
}
typedef uint8_t __attribute__((address_space(3))) LdsBytes;

// What a launch keeps of its circuit at the start of the dynamic LDS: the
// truncation statistics, read from and written to global memory once per
// launch (a read-modify-write in every step would hold up its end).
struct CircuitLds {
  double disc, maxdisc;
  int degen, unconv;
  int64_t unused;
};

template <typename T>
__device__ inline T *lds_at(int offset) {
  return reinterpret_cast<T *>((uint8_t *)(LdsBytes *)(uintptr_t)uniform(offset));
}

constexpr int kKC = 16;  // contraction chunk of the pair product staged in LDS

// Two-site steps are compiled for Jacobi matrices up to N x N (N = 16, 32,
// 64, 128) in workgroups of W waves, of which WA hold the matrix.  A wave's
// lanes are N / 2 column pairs (lane cp of a row group holds column positions
// 2 cp and 2 cp + 1) times RG row groups of ROWS rows, so small matrices fill
// the lanes, and one wave needs neither LDS round trips nor barriers between
// its rows and columns.  More waves than WA only lengthen the rounds of a
// small matrix: each reads the round's sums from LDS.
template <int N, int W>
struct Layout {
  static constexpr int WA = N == 32 ? (W < 4 ? W : 4) : N == 64 ? (W < 8 ? W : 8) : W;
  static constexpr int LC = N / 2;                 // column pairs
  static constexpr int RG = 64 / LC;               // row groups of a wave
  static constexpr int GR = WA * RG;               // row groups of the matrix
  static constexpr int ROWS = N > GR ? N / GR : 1; // rows per group
  static constexpr int HROWS = N / 2 > GR ? N / 2 / GR : 1;   // of a block of N / 2 rows
  static constexpr int SLOTS = GR * ROWS;
  static constexpr int T = 64 * W;
  static constexpr bool kLds = N <= 32;            // pair product and isometry in LDS
  // rotations of a round: formed by every wave for its own lanes from the
  // waves' partial sums, or (N = 128, where every wave would read 16 of them
  // for each of 64 pairs) by four waves and read back
  static constexpr bool kOwn = N <= 64;
};

// Barrier of the W waves that run a step; with one wave, its own order (LDS
// and memory accesses of one wave take effect in program order, so nothing
// waits for the stores).
template <int W>
__device__ inline void step_sync() {
  if constexpr (W == 1) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

template <int N, int W>
struct StepLds {
  using Y = Layout<N, W>;
  union {
    struct {
      double2 L[kKC][Y::SLOTS];
      double2 R[kKC][N];
    } stage;                       // contraction chunks (dead once the Jacobi matrix is built)
    double2 red[2][2][Y::WA][Y::LC];   // per round type: (|X|^2, |Y|^2) and <X, Y> by wave and pair
    double2 U[Y::kLds ? N * N : 1];// isometry (row-major), after the sweeps
  };
  double2 P2[Y::kLds ? N * N : 1]; // pair product
  double2 lqw[N];                  // Householder vector of an LQ step
  double rot[2][3][Y::kOwn ? 1 : Y::LC + 1];   // per round type: c, sigma of pair p at p + 1 (N = 128)
  double w[N];                     // row norms during the LQ, then (N = 128) column norms by position
  double norm[N], sorted[N];
  double part[W];
  double beta, nrm;
  int flag;
  int rank[N];
  int k;
};

// s and a of a combined index s D + a, s in {0, 1}
__device__ inline int phys_of(int x, int D) { return x >= D ? 1 : 0; }

// Sum over the LC lanes of a row group (every lane receives the total).
template <int LC>
__device__ inline double cols_sum(double x) {
  if constexpr (LC == 8) {
    x += dpp_mov<0xB1>(x);    // quad_perm [1,0,3,2]
    x += dpp_mov<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_mov<0x141>(x);   // row_half_mirror: the other quad of eight lanes
  } else {
    x = row_sum16(x);
    if constexpr (LC >= 32) {
      double y = x;
      swap16(x, y);
      x += y;
    }
    if constexpr (LC == 64) {
      double y = x;
      swap32(x, y);
      x += y;
    }
  }
  return x;
}

// Sum over the row groups of a wave (every lane receives its column's).
template <int LC>
__device__ inline double groups_sum(double x) {
  if constexpr (LC == 8) x += dpp_mov<0x128>(x);   // row_ror:8
  if constexpr (LC <= 16) {
    double y = x;
    swap16(x, y);
    x += y;
  }
  if constexpr (LC <= 32) {
    double y = x;
    swap32(x, y);
    x += y;
  }
  return x;
}

// Block-wide complex product acc[rr][q] = sum_{k < K} L(y, k) R(k, x) with
// y = NR (row group) + rr and x = 2 cp + q; ldL / ldR return the operands
// (zero outside the matrices).  Chunks of kKC contraction indices of both
// operands are staged in LDS.
template <int N, int W, int NR, class FL, class FR>
__device__ inline void staged_tile_gemm(int K, const FL &ldL, const FR &ldR, StepLds<N, W> &sh,
                                        double2 (&acc)[NR][2]) {
  using Y = Layout<N, W>;
  const int tid = W == 1 ? threadIdx.x & 63 : threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cp = lane % Y::LC, y0 = (wave * Y::RG + lane / Y::LC) * NR;
  constexpr int kRowsAll = NR * Y::GR;
#pragma unroll
  for (int rr = 0; rr < NR; ++rr) {
    acc[rr][0] = make_double2(0.0, 0.0);
    acc[rr][1] = make_double2(0.0, 0.0);
  }
  for (int k0 = 0; k0 < K; k0 += kKC) {
    step_sync<W>();  // the previous chunk (or earlier use of the buffers) is done
    // every load of the chunk is in flight before the first is stored
    constexpr int NL = (kKC * kRowsAll + Y::T - 1) / Y::T, NR2 = (kKC * N + Y::T - 1) / Y::T;
    double2 vl[NL], vr[NR2];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      // consecutive threads walk the contraction index of one row
      const int e = tid + u * Y::T, kk = e % kKC, y = e / kKC;
      vl[u] = y < kRowsAll && k0 + kk < K ? ldL(y, k0 + kk) : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < NR2; ++u) {
      const int e = tid + u * Y::T, x = e % N, kk = e / N;
      vr[u] = kk < kKC && k0 + kk < K ? ldR(k0 + kk, x) : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int u = 0; u < NL; ++u) {
      const int e = tid + u * Y::T;
      if (e < kKC * kRowsAll) sh.stage.L[e % kKC][e / kKC] = vl[u];
    }
#pragma unroll
    for (int u = 0; u < NR2; ++u) {
      const int e = tid + u * Y::T;
      if (e < kKC * N) sh.stage.R[e / N][e % N] = vr[u];
    }
    step_sync<W>();
    const int kc = wave < Y::WA ? min(kKC, K - k0) : 0;
    for (int kk = 0; kk < kc; ++kk) {
      const double2 r0 = sh.stage.R[kk][2 * cp], r1 = sh.stage.R[kk][2 * cp + 1];
#pragma unroll
      for (int rr = 0; rr < NR; ++rr) {
        const double2 l = sh.stage.L[kk][y0 + rr];
        acc[rr][0].x = fma(l.x, r0.x, fma(-l.y, r0.y, acc[rr][0].x));
        acc[rr][0].y = fma(l.x, r0.y, fma(l.y, r0.x, acc[rr][0].y));
        acc[rr][1].x = fma(l.x, r1.x, fma(-l.y, r1.y, acc[rr][1].x));
        acc[rr][1].y = fma(l.x, r1.y, fma(l.y, r1.x, acc[rr][1].y));
      }
    }
  }
}

// Two-site theta element theta[(s, a), (t, b)] of this step's gate from the
// pair product P (row stride ld).
__device__ inline double2 theta_from_pair(const double2 *Pp2, int op, double cg, double sg, int Dp, int Dn, int s,
                                          int a, int t, int b, int ld) {
  if (op == OP_SWAP) return Pp2[(t * Dp + a) * ld + s * Dn + b];
  const double2 d = Pp2[(s * Dp + a) * ld + t * Dn + b];
  if (op == OP_RXX) {
    // Rxx = cos(phi/2) I - i sin(phi/2) X(x)X
    const double2 x = Pp2[((1 - s) * Dp + a) * ld + (1 - t) * Dn + b];
    return make_double2(cg * d.x + sg * x.y, cg * d.y - sg * x.x);
  }
  return d;
}

// Sum over the 4 lanes of a DPP quad (every lane receives the same total).
__device__ inline double quad_sum(double x) {
  x += dpp_mov<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp_mov<0x4E>(x);   // quad_perm [2,3,0,1]
  return x;
}

// Rotation of a column pair (X, Y) with squared norms a, b and <X, Y> = g:
// X' = c X - sigma Y, Y' = conj(sigma) X + c Y (the Hermitian 2 x 2 Jacobi
// rotation of the pair's Gram block up to the phase of Y') zeroes <X', Y'>.
// With p = b - a and h = sqrt(p^2 + 4 |g|^2): c^2 = (1 + |p| / h) / 2 and
// sigma = sign(p) conj(g) / (h c), two dependent reciprocal square roots in
// all (this chain is the longest part of a round's latency).  tg: the amount
// by which |Y'|^2 exceeds b and |X'|^2 falls below a.
struct Rotation {
  double c, sr, si, tg;
};
__device__ inline Rotation rotation(double a, double b, double x, double y, double g2) {
  const double p = b - a;
  const double rh = rsqrt(fma(p, p, 4.0 * g2));
  const double c2 = fma(0.5 * fabs(p), rh, 0.5);
  const double rc = rsqrt(c2);
  const double f = p >= 0.0 ? rh : -rh;
  Rotation r;
  r.c = c2 * rc;
  const double frc = f * rc;
  r.sr = x * frc;
  r.si = -y * frc;
  r.tg = g2 * frc * rc;
  return r;
}

// One round of the parallel Jacobi sweep.  The pair of a lane is (X, Y) =
// (A, B) for TYPE 0 and (B_l, A_{l+1}) for TYPE 1; the rotated columns are
// stored exchanged, Y' in the slot of X and X' in the slot of Y: with the
// pair's (c, sigma), TYPE 0 forms A' = c B + conj(sigma) A, B' = c A - sigma B,
// TYPE 1 B' = c A_{l+1} + conj(sigma) B and, with the pair of lane l - 1,
// A' = c B_{l-1} - sigma A.  Where there is no pair, (0, 1) keeps the column
// up to its sign.  Returns whether some pair seen by this wave was rotated by
// more than kJacobiLarge (relative |<X,Y>|).
//
// Column norms: a FULL round reduces |X|^2 and |Y|^2 with <X, Y> and stores
// them; the other rounds reduce <X, Y> only and update the stored norms by
// |X'|^2 = |X|^2 - t |<X,Y>|, |Y'|^2 = |Y|^2 + t |<X,Y>| (t = s / c), which
// holds exactly for the rotation above.  The first round of every sweep is
// FULL, so rounding in the updates never outlives a sweep.
//
// A round is a chain of dependent FP64 operations (~24 cycles each), LDS
// accesses and barriers.  Up to 64 x 64 every wave adds up the partial sums
// and forms the rotations of its own lanes (identical in all waves), which
// takes one barrier; with four waves forming them for all, two barriers and
// conflicting reads of the results, a 64 x 64 round took 3,700 cycles and a
// 32 x 32 one 4,600 (16 waves).
template <int N, int W>
struct Columns {
  static constexpr int ROWS = Layout<N, W>::ROWS;
  double Ar[ROWS], Ai[ROWS], Br[ROWS], Bi[ROWS];
  double wA, wB;   // squared norms (kOwn)
};

template <int N, int W, int TYPE, bool FULL>
__device__ __forceinline__ bool jacobi_round(Columns<N, W> &M, StepLds<N, W> &sh, int wave, int H, double zero_w) {
  using Y = Layout<N, W>;
  constexpr int ROWS = Y::ROWS, LC = Y::LC, WA = Y::WA;
  // The lane index is formed afresh every round (two instructions the
  // compiler cannot hoist), so the LDS addresses derived from it are not
  // held, or spilled, across the sweep loop.
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  const int cp = lane & (LC - 1);
  const int npairs = TYPE == 0 ? H : H - 1;
  bool large = false;
  double Nr[ROWS], Ni[ROWS];  // A_{l+1} (TYPE 1)
  double al = 0.0, be = 0.0, gr = 0.0, gi = 0.0;
  if (WA == W || wave < WA) {
    if (TYPE == 1) {
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr) {
        Nr[rr] = dpp_shl1(M.Ar[rr]);
        Ni[rr] = dpp_shl1(M.Ai[rr]);
      }
    }
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) {
      const double xr = TYPE == 0 ? M.Ar[rr] : M.Br[rr], xi = TYPE == 0 ? M.Ai[rr] : M.Bi[rr];
      const double yr = TYPE == 0 ? M.Br[rr] : Nr[rr], yi = TYPE == 0 ? M.Bi[rr] : Ni[rr];
      if (FULL) {
        al = fma(xr, xr, fma(xi, xi, al));
        be = fma(yr, yr, fma(yi, yi, be));
      }
      gr = fma(xr, yr, fma(xi, yi, gr));
      gi = fma(xr, yi, fma(-xi, yr, gi));
    }
    if constexpr (W > 1 && Y::kOwn) {
      // partial sums of the wave: lane rows (halves) 0 end with the first
      // value of a pair, the upper half with the second
      auto put = [&](double2 &slot, double x, double y) {
        swap32(x, y);
        x += y;
        if constexpr (Y::RG == 4) {
          double z = x;
          swap16(x, z);
          x += z;
        }
        if (Y::RG == 2 || (lane & 16) == 0) (lane < 32 ? slot.x : slot.y) = x;
      };
      if (FULL) put(sh.red[TYPE][0][wave][cp], al, be);
      put(sh.red[TYPE][1][wave][cp], gr, gi);
    } else if constexpr (W > 1) {
      if (FULL) sh.red[0][0][wave][cp] = make_double2(al, be);
      sh.red[0][1][wave][cp] = make_double2(gr, gi);
    }
  }
  if constexpr (W > 1) __syncthreads();
  double c = 0.0, sr = 1.0, si = 0.0;      // of the lane's pair
  double cp_ = 0.0, srp = 1.0, sip = 0.0;  // of the pair of lane l - 1 (TYPE 1)
  if constexpr (Y::kOwn) {
    if (WA < W && wave >= WA) return false;
    double a = 0.0, b = 0.0;
    if constexpr (W == 1) {
      gr = groups_sum<LC>(gr);
      gi = groups_sum<LC>(gi);
      if (FULL) {
        a = groups_sum<LC>(al);
        b = groups_sum<LC>(be);
      }
    } else {
      // row group rg adds the partials of waves rg, rg + RG, ..., then the
      // row groups together
      auto get = [&](const double2 (*red)[LC], double &x, double &y) {
        x = y = 0.0;
#pragma unroll
        for (int u = 0; u < WA / Y::RG; ++u) {
          const double2 v = red[lane / LC + u * Y::RG][cp];
          x += v.x;
          y += v.y;
        }
        x = groups_sum<LC>(x);
        y = groups_sum<LC>(y);
      };
      get(sh.red[TYPE][1], gr, gi);
      if (FULL) get(sh.red[TYPE][0], a, b);
    }
    if (!FULL) {
      a = TYPE == 0 ? M.wA : M.wB;
      b = TYPE == 0 ? M.wB : dpp_shl1(M.wA);
    }
    const double g2 = fma(gr, gr, gi * gi);
    const bool act = cp < npairs;
    const bool rot = act && a > zero_w && b > zero_w && g2 > (kJacobiTol * kJacobiTol) * (a * b);
    large = rot && g2 > (kJacobiLarge * kJacobiLarge) * (a * b);
    double tg = 0.0;
    if (act) {
      c = 1.0;
      sr = 0.0;
    }
    if (rot) {
      const Rotation r = rotation(a, b, gr, gi, g2);
      c = r.c;
      sr = r.sr;
      si = r.si;
      tg = r.tg;
    }
    const double nX = b + tg, nY = fmax(a - tg, 0.0);   // exchanged: norms of the slots of X and Y
    if (TYPE == 0) {
      if (act) {
        M.wA = nX;
        M.wB = nY;
      }
    } else {
      cp_ = dpp_shr1(c);   // 0 for the first pair's A, which has no partner (the lane before holds none)
      srp = dpp_shr1(sr);
      sip = dpp_shr1(si);
      const double na = dpp_shr1(nY);
      if (cp == 0) srp = 1.0;
      if (act) M.wB = nX;
      if (cp > 0 && cp <= npairs) M.wA = na;
    }
  } else {
    // lane = 4 j + q of the first waves sums the partials of pair
    // 16 wave + j over waves W/4 q .. W/4 (q + 1) - 1, then over the quad
    if (16 * wave < npairs) {
      const int j = lane >> 2, q = lane & 3, pr = 16 * wave + j;
      // positions of X and Y
      const int px = TYPE == 0 ? 2 * pr : 2 * pr + 1, py = px + 1;
      double a = 0.0, b = 0.0, x = 0.0, y = 0.0;
#pragma unroll
      for (int u = 0; u < W / 4; ++u) {
        if (FULL) {
          const double2 n = sh.red[0][0][W / 4 * q + u][pr];
          a += n.x;
          b += n.y;
        }
        const double2 g = sh.red[0][1][W / 4 * q + u][pr];
        x += g.x;
        y += g.y;
      }
      if (FULL) {
        a = quad_sum(a);
        b = quad_sum(b);
      } else {
        a = sh.w[px];
        b = sh.w[py < N ? py : N - 1];
      }
      x = quad_sum(x);
      y = quad_sum(y);
      const double g2 = fma(x, x, y * y);
      const bool rot = pr < npairs && a > zero_w && b > zero_w && g2 > (kJacobiTol * kJacobiTol) * (a * b);
      large = rot && g2 > (kJacobiLarge * kJacobiLarge) * (a * b);
      if (pr < npairs && q == 0) {
        Rotation r{1.0, 0.0, 0.0, 0.0};
        if (rot) r = rotation(a, b, x, y, g2);
        // exchanged: the slot of X receives |Y'|^2, the slot of Y |X'|^2
        sh.w[px] = b + r.tg;
        sh.w[py] = fmax(a - r.tg, 0.0);
        sh.rot[TYPE][0][pr + 1] = r.c;
        sh.rot[TYPE][1][pr + 1] = r.sr;
        sh.rot[TYPE][2][pr + 1] = r.si;
      }
    }
    __syncthreads();
    c = sh.rot[TYPE][0][cp + 1];
    sr = sh.rot[TYPE][1][cp + 1];
    si = sh.rot[TYPE][2][cp + 1];
    if (TYPE == 1) {
      cp_ = sh.rot[TYPE][0][cp];
      srp = sh.rot[TYPE][1][cp];
      sip = sh.rot[TYPE][2][cp];
    }
  }
#pragma unroll
  for (int rr = 0; rr < ROWS; ++rr) {
    const double ar = M.Ar[rr], ai = M.Ai[rr], br = M.Br[rr], bi = M.Bi[rr];
    if (TYPE == 0) {
      M.Ar[rr] = fma(c, br, fma(sr, ar, si * ai));
      M.Ai[rr] = fma(c, bi, fma(sr, ai, -si * ar));
      M.Br[rr] = fma(c, ar, fma(-sr, br, si * bi));
      M.Bi[rr] = fma(c, ai, fma(-sr, bi, -si * br));
    } else {
      const double pr_ = dpp_shr1(br), pi_ = dpp_shr1(bi);
      M.Br[rr] = fma(c, Nr[rr], fma(sr, br, si * bi));
      M.Bi[rr] = fma(c, Ni[rr], fma(sr, bi, -si * br));
      M.Ar[rr] = fma(cp_, pr_, fma(-srp, ar, sip * ai));
      M.Ai[rr] = fma(cp_, pi_, fma(-srp, ai, -sip * ar));
    }
  }
  return large;
}

// One entry of the step list shared by every circuit of a batch: a run of
// Rz records, or a two-site step (a two-qubit gate or a centre move).
enum StepKind { STEP_RZ = 0, STEP_TWO_SITE = 1 };
struct SimStep {
  int32_t kind;
  int32_t p, mode, op, fi, fj;  // two-site step: sites (p, p+1), SvMode, GateOp, features of Rxx
  int32_t r0;                   // Rz run: first gate record; two-site step: index of the two-qubit
                                // gate among the circuit's (-1 for a centre move)
  int32_t nr;                   // Rz run: gate records [r0, r0 + nr); two-site step: largest bond
                                // that can result (the kernel is chosen for these)
  int32_t Pp, Pm, Pn;           // two-site step: pads of the three bonds, and the offsets of both
  int32_t unused;               // sites in an MPS (with the step, so that no step waits for them)
  int64_t off_p, off_q;
};

// Largest row norm of the rows that are no pivot yet: the sign-less upper
// halves order like the norms; the low bits carry the row (complemented).
template <int N>
__device__ inline int heaviest_row(const double *rn, int lane) {
  constexpr uint32_t kRow = N > 128 ? 255 : 127;
  uint32_t best = 0;
#pragma unroll
  for (int u = 0; u < (N + 63) / 64; ++u) {
    const int row = lane + 64 * u;
    const double v = row < N ? rn[row] : -1.0;
    const uint32_t key = v < 0.0 ? 0u : (uint32_t(__double2hiint(v)) & ~kRow) | (kRow - row);
    best = max(best, key);
  }
  return int(kRow - (wave_max_bits(best) & kRow));
}

// Squared norms of the rows of M (row r < N to sh.w, -1 beyond nr) and
// ||M||_F^2, in every lane.
template <int N, int W>
__device__ __forceinline__ double row_weights(const Columns<N, W> &M, StepLds<N, W> &sh, int nr, int tid) {
  using Y = Layout<N, W>;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cp = lane % Y::LC, row0 = (wave * Y::RG + lane / Y::LC) * Y::ROWS;
  double tot = 0.0;
#pragma unroll
  for (int rr = 0; rr < Y::ROWS; ++rr) {
    const int r = row0 + rr;
    const double n2 = fma(M.Ar[rr], M.Ar[rr], fma(M.Ai[rr], M.Ai[rr], fma(M.Br[rr], M.Br[rr], M.Bi[rr] * M.Bi[rr])));
    tot += n2;
    const double rn = cols_sum<Y::LC>(n2);
    if (cp == 0 && r < N) sh.w[r] = r < nr ? rn : -1.0;
  }
  tot = wave_sum(tot);
  if constexpr (W > 1) {
    if (lane == 0) sh.part[wave] = tot;
    __syncthreads();
    tot = 0.0;
#pragma unroll
    for (int u = 0; u < W; ++u) tot += sh.part[u];
  }
  step_sync<W>();
  return tot;
}

// LQ preconditioning of M (nr rows, nref = min(rows, columns) reflections);
// sh.w holds the rows' squared norms.
//
// M <- M H_0 H_1 ... (Householder reflections from the right, M = L Q with
// the heaviest remaining row as the next pivot): the Jacobi columns of
// M W are U S for any unitary W, so the factors are unchanged, while the
// triangular factor of these graded matrices needs half the sweeps of M
// itself and only its first min(nr, nc) columns carry more than rounding.
// Step i reflects its pivot row onto column i: with x = that row restricted
// to columns >= i and w = x + e^{i arg x_i} |x| e_i, every row r becomes
// r - beta (r . conj w) w, beta = 1 / (|x| (|x| + |x_i|)).  Rows stay in
// place (a row permutation changes no column inner product); their
// remaining norms are reduced by each new entry.  128 x 128 thetas of a
// d = 8 circuit: 7.7 sweeps against 8.7 with the rows in order of initial
// norm (30 x 64 ones of a d = 3 circuit: 6.6 against 7.3).
template <int N, int W>
__device__ __forceinline__ void lq_reduce(Columns<N, W> &M, StepLds<N, W> &sh, int nr, int nref, int tid) {
  using Y = Layout<N, W>;
  constexpr int ROWS = Y::ROWS, LC = Y::LC;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cp = lane % LC, row0 = (wave * Y::RG + lane / LC) * ROWS;
  const int c0 = 2 * cp, c1 = 2 * cp + 1;
  constexpr bool kSkip = N >= 64;   // the branches cost small matrices more than the rows
  // Bits 4 rr .. of `fin`: how many row groups of this wave have row rr done (a
  // pivot, or beyond nr); a row that all have done is left out of the updates
  // (128 x 128: 520,000 -> 463,000 cycles per LQ)
  uint32_t fin = 0;
  if constexpr (kSkip) {
#pragma unroll
    for (int g = 0; g < Y::RG; ++g)
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr) fin += (wave * Y::RG + g) * ROWS + rr < nr ? 0u : 1u << (4 * rr);
  }
  constexpr uint32_t kAll = 0x11111111u * Y::RG & uint32_t((1ull << (4 * ROWS)) - 1);
  for (int i = 0; i < nref; ++i) {
    const uint32_t before = fin;
    const int pv = __builtin_amdgcn_readfirstlane(heaviest_row<N>(sh.w, lane));
    const int pg = pv / ROWS, ri = pv % ROWS;   // row group and row of the pivot
    if (wave == pg / Y::RG) {
      fin += 1u << (4 * ri);
      double xr0 = 0.0, xi0 = 0.0, xr1 = 0.0, xi1 = 0.0;
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr)
        if (rr == ri) {
          xr0 = M.Ar[rr];
          xi0 = M.Ai[rr];
          xr1 = M.Br[rr];
          xi1 = M.Bi[rr];
        }
      if (c0 < i) xr0 = xi0 = 0.0;
      if (c1 < i) xr1 = xi1 = 0.0;
      const double n2 = cols_sum<LC>(fma(xr0, xr0, fma(xi0, xi0, fma(xr1, xr1, xi1 * xi1))));
      if (lane / LC == pg % Y::RG) {
        const double dr = (i & 1) ? xr1 : xr0, di = (i & 1) ? xi1 : xi0;
        const double a2 = fma(dr, dr, di * di);
        const double rn = n2 > 0.0 ? rsqrt(n2) : 0.0, ra = a2 > 0.0 ? rsqrt(a2) : 0.0;
        const double nx = n2 * rn, ax = a2 * ra;
        const double pr = a2 > 0.0 ? dr * ra : 1.0, pi = di * ra;
        const double2 d = make_double2(pr * (ax + nx), pi * (ax + nx));
        sh.lqw[c0] = c0 == i ? d : make_double2(xr0, xi0);
        sh.lqw[c1] = c1 == i ? d : make_double2(xr1, xi1);
        if (cp == (i >> 1)) sh.beta = n2 > 0.0 ? rn * reciprocal(nx + ax) : 0.0;
      }
    }
    step_sync<W>();
    if (wave < Y::WA && before != kAll) {
      const double2 w0 = sh.lqw[c0], w1 = sh.lqw[c1];
      const double beta = sh.beta;
      double d[2 * ROWS];  // d = r . conj(w) for the rows (re, im)
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr) {
        d[2 * rr] = d[2 * rr + 1] = 0.0;
        if (kSkip && ((before >> (4 * rr)) & 15u) == Y::RG) continue;
        d[2 * rr] = fma(M.Ar[rr], w0.x, fma(M.Ai[rr], w0.y, fma(M.Br[rr], w1.x, M.Bi[rr] * w1.y)));
        d[2 * rr + 1] = fma(M.Ai[rr], w0.x, fma(-M.Ar[rr], w0.y, fma(M.Bi[rr], w1.x, -M.Br[rr] * w1.y)));
      }
      if constexpr (LC == 64 && ROWS == 8) {
        wave_sum16(d);
      } else if constexpr (LC == 32 && ROWS == 8) {
        half_sum16(d);
      } else {
#pragma unroll
        for (int u = 0; u < 2 * ROWS; ++u) d[u] = cols_sum<LC>(d[u]);
      }
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr) {
        if (kSkip && ((before >> (4 * rr)) & 15u) == Y::RG) continue;
        const double dr = beta * d[2 * rr], di = beta * d[2 * rr + 1];
        M.Ar[rr] -= dr * w0.x - di * w0.y;
        M.Ai[rr] -= dr * w0.y + di * w0.x;
        M.Br[rr] -= dr * w1.x - di * w1.y;
        M.Bi[rr] -= dr * w1.y + di * w1.x;
        if (cp == (i >> 1) && row0 + rr < nr) {
          const double er = (i & 1) ? M.Br[rr] : M.Ar[rr], ei = (i & 1) ? M.Bi[rr] : M.Ai[rr];
          const double v = sh.w[row0 + rr];
          sh.w[row0 + rr] = row0 + rr == pv || v < 0.0 ? -1.0 : fmax(v - fma(er, er, ei * ei), 0.0);
        }
      }
      if (kSkip && wave == pg / Y::RG) {   // the pivot row ends at column i
#pragma unroll
        for (int rr = 0; rr < ROWS; ++rr)
          if (rr == ri && lane / LC == pg % Y::RG) {
            if (c0 > i) M.Ar[rr] = M.Ai[rr] = 0.0;
            if (c1 > i) M.Br[rr] = M.Bi[rr] = 0.0;
          }
      }
    }
    step_sync<W>();
  }
}

// One-sided Jacobi sweeps over the first 2 H columns of M; returns whether
// they converged.
//
// Odd-even transposition ordering of the positions 0..2H-1 (A_l = 2l,
// B_l = 2l+1): type-0 rounds pair (A_l, B_l) inside each lane, type-1 rounds
// pair (B_l, A_{l+1}) across neighbouring lanes, and each pair is exchanged
// after its rotation, so every two columns meet exactly once in the 2H rounds
// of a sweep.  Positions beyond keep what they hold.
template <int N, int W>
__device__ __forceinline__ bool jacobi_sweeps(Columns<N, W> &M, StepLds<N, W> &sh, int H, double zero_w, int tid) {
  using Y = Layout<N, W>;
  constexpr int LC = Y::LC;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if constexpr (!Y::kOwn) {
    // pairs that no round of the type has
    for (int e = tid; e < 2 * (LC + 1); e += Y::T) {
      const int type = e / (LC + 1), x = e % (LC + 1);
      sh.rot[type][0][x] = sh.rot[type][2][x] = 0.0;
      sh.rot[type][1][x] = 1.0;
    }
    __syncthreads();
  }
  bool converged = false;
  for (int sweep = 0; sweep < kMaxSweeps && !converged; ++sweep) {
    bool large = jacobi_round<N, W, 0, true>(M, sh, wave, H, zero_w);
    if (H > 1) large |= jacobi_round<N, W, 1, false>(M, sh, wave, H, zero_w);
    for (int half = 1; half < H; ++half) {
      large |= jacobi_round<N, W, 0, false>(M, sh, wave, H, zero_w);
      large |= jacobi_round<N, W, 1, false>(M, sh, wave, H, zero_w);
    }
    if constexpr (W == 1) {
      converged = __any(large) == 0;
    } else {
      // large is known to wave 0 (kOwn) or to each of the first four waves
      if (tid == 0) sh.flag = 0;
      __syncthreads();
      if (large) sh.flag = 1;
      __syncthreads();
      converged = uniform(sh.flag) == 0;
    }
  }
  return converged;
}

// Norms, order and number of the columns kept (Eq. (8)) after the sweeps:
// sh.norm by position, sh.rank, sh.k and the factor sh.nrm that restores unit
// weight; the truncation statistics of the circuit.
template <int N, int W>
__device__ __forceinline__ void select_columns(const Columns<N, W> &M, StepLds<N, W> &sh, CircuitLds &cl,
                                               const SvParams &P, const SimStep &st, bool gate, double cg, double sg, int Dm,
                                               int nref, int NP, double zero_w, bool converged, int tid) {
  using Y = Layout<N, W>;
  constexpr int ROWS = Y::ROWS, LC = Y::LC;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cp = lane % LC, c0 = 2 * cp, c1 = 2 * cp + 1;
  double na = 0.0, nb = 0.0;
#pragma unroll
  for (int rr = 0; rr < ROWS; ++rr) {
    na = fma(M.Ar[rr], M.Ar[rr], fma(M.Ai[rr], M.Ai[rr], na));
    nb = fma(M.Br[rr], M.Br[rr], fma(M.Bi[rr], M.Bi[rr], nb));
  }
  na = groups_sum<LC>(na);
  nb = groups_sum<LC>(nb);
  if constexpr (W > 1) {
    if (wave < Y::WA && lane < LC) sh.red[0][0][wave][cp] = make_double2(na, nb);
    __syncthreads();
    if (tid < LC) {
      na = nb = 0.0;
#pragma unroll 4
      for (int u = 0; u < Y::WA; ++u) {
        na += sh.red[0][0][u][tid].x;
        nb += sh.red[0][0][u][tid].y;
      }
    }
  }
  if (tid < LC) {
    sh.norm[c0] = c0 < NP ? na : 0.0;
    sh.norm[c1] = c1 < NP ? nb : 0.0;
  }
  step_sync<W>();
  if (tid < 4 * N) {
    // four threads per position count the columns that precede it
    const int pos = tid >> 2;
    const double v = sh.norm[pos];
    int rank = 0;
#pragma unroll 8
    for (int u = 0; u < N / 4; ++u) {
      const int x = 4 * u + (tid & 3);
      const double o = sh.norm[x];
      rank += (o > v || (o == v && x < pos)) ? 1 : 0;
    }
    rank += __builtin_amdgcn_mov_dpp(rank, 0xB1, 0xf, 0xf, true);
    rank += __builtin_amdgcn_mov_dpp(rank, 0x4E, 0xf, 0xf, true);
    if ((tid & 3) == 0) {
      sh.rank[pos] = rank;
      sh.sorted[rank] = v;
    }
  }
  step_sync<W>();
  if (wave == 0) {
    // lane l holds the sorted weights PER l .. PER l + PER - 1 and, in suf,
    // the weight from each on
    constexpr int PER = N > 64 ? N / 64 : 1;
    double v[PER], suf[PER], s = 0.0;
#pragma unroll
    for (int u = PER - 1; u >= 0; --u) {
      v[u] = PER * lane + u < N ? sh.sorted[PER * lane + u] : 0.0;
      s += v[u];
      suf[u] = s;
    }
    double rest;
    if constexpr (N == 16) {   // within the first row of lanes (the others hold zeros)
      s += dpp_mov<0x101>(s);  // row_shl
      s += dpp_mov<0x102>(s);
      s += dpp_mov<0x104>(s);
      s += dpp_mov<0x108>(s);
      rest = dpp_mov<0x101>(s);
    } else {
#pragma unroll
      for (int o = 1; o < 64 && o * PER < N; o <<= 1) {
        const double t = __shfl_down(s, o, 64);
        s += lane + o < 64 ? t : 0.0;
      }
      rest = __shfl_down(s, 1, 64);
    }
    const double total = lane0(s);
    int nnz = 0, above = 0;
    const int nsv = nref;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      suf[u] += lane < 63 ? rest : 0.0;
      const bool in = PER * lane + u < nsv;
      nnz += __popcll(__ballot(PER * lane + u < N && v[u] > zero_w));
      above += __popcll(__ballot(in && suf[u] > P.cutoff * total));
    }
    int k;
    double nrm = 1.0;
    if (gate) {
      // smallest k with sum_{r >= k} w_r <= cutoff * total
      const int kcut = P.cutoff > 0.0 ? above : nsv;
      k = max(1, min(min(P.chi, kcut), max(nnz, 1)));
      if (P.gate_split) {
        // theta = sum_r (L_r A_p)(R_r A_{p+1}) over the rank(G) terms of
        // the gate's operator-Schmidt decomposition: rank <= rank(G) Dm.
        // Rxx(phi) = cos(phi/2) II - i sin(phi/2) XX: a term counts when its
        // coefficient exceeds 1e-12 of the larger one (cos(pi/2) rounds to
        // ~6e-17, not zero); SWAP has four terms
        const double cmax = fmax(fabs(cg), fabs(sg));
        const int rg = st.op == OP_RXX
                           ? (fabs(cg) > 1e-12 * cmax ? 1 : 0) + (fabs(sg) > 1e-12 * cmax ? 1 : 0)
                           : 4;
        k = max(1, min(k, rg * Dm));
      }
      k = min(k, st.nr);
      k = uniform(k);
      // weight of the columns left out: the suffix sum from column k on
      double tail = 0.0;
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const double t = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(suf[u]), (k / PER) & 63),
                                          __builtin_amdgcn_readlane(__double2loint(suf[u]), (k / PER) & 63));
        if (k < N && k % PER == u) tail = t;
      }
      const double kept = total - tail;
      nrm = kept > 0.0 ? rsqrt(kept) : 1.0;
      if (lane == 0) {
        const double disc = total > 0.0 ? tail * reciprocal(total) : 0.0;
        cl.disc += disc;
        cl.maxdisc = fmax(cl.maxdisc, disc);
        // (sqrt(w_k-1) - sqrt(w_k)) / sqrt(w_0) below the gap: the difference
        // of the roots is at least that of the weights over 2 sqrt(w_k-1)
        if (k < nsv && sh.sorted[0] > 0.0) {
          const double wa = sh.sorted[k - 1], wb = sh.sorted[k], w0 = sh.sorted[0];
          if ((wa - wb) * (wa - wb) <= (8.0 * kDegenerateGap * kDegenerateGap) * (wa * w0) &&
              (sqrt(wa) - sqrt(wb)) / sqrt(w0) < kDegenerateGap)
            cl.degen += 1;
        }
      }
    } else {
      k = min(max(1, min(nsv, max(nnz, 1))), st.nr);
    }
    if (lane == 0) {
      if (!converged) cl.unconv += 1;
      sh.k = k;
      sh.nrm = nrm;
    }
  }
  step_sync<W>();
}

// Two-site step of circuit ci on W waves, for Jacobi matrices up to N x N.
template <int N, int W>
__device__ __attribute__((noinline)) void svd_step(const SvParams *Pp, int64_t ci_, const SimStep *stp,
                                                   int lds, int Dp_, int Dm_, int Dn_) {
  using Y = Layout<N, W>;
  constexpr int ROWS = Y::ROWS, LC = Y::LC;
  CircuitLds &cl = *lds_at<CircuitLds>(lds);
  StepLds<N, W> &sh = *lds_at<StepLds<N, W>>(lds + int(sizeof(CircuitLds)));
  const SvParams P = uniform_load(Pp);
  const SimStep st = uniform_load(stp);
  const int64_t ci = uniform(ci_);
  const int tid = W == 1 ? threadIdx.x & 63 : threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar register
  const int cp = lane % LC, row0 = (wave * Y::RG + lane / LC) * ROWS;
  const int c0 = 2 * cp;

  int32_t *dims = P.dims + ci * (P.m + 1);
  const int p = st.p;
  const int Dp = uniform(Dp_), Dm = uniform(Dm_), Dn = uniform(Dn_);
  const int Pw = st.Pp, Pm = st.Pm, Pn = st.Pn;
  double2 *Ap = P.f64 + ci * P.mps_stride + st.off_p;
  double2 *Aq = P.f64 + ci * P.mps_stride + st.off_q;
  double2 *P2 = Y::kLds ? sh.P2 : P.scratch + int64_t(blockIdx.x) * P.scratch_stride;

  double cg = 1.0, sg = 0.0;
  if (st.op == OP_RXX) {
    const double xi = P.X[ci * P.ldx + st.fi], xj = P.X[ci * P.ldx + st.fj];
    const double phi = P.coef_xx * (1.0 - xi) * (1.0 - xj);
    sincos(0.5 * phi, &sg, &cg);
  }

  const bool right = (st.mode == GATE_RIGHT || st.mode == MOVE_RIGHT);
  const bool gate = (st.mode == GATE_RIGHT || st.mode == GATE_LEFT);
  // Jacobi matrix shape and projection-source width
  int nr, nc, ncs;
  if (st.mode == GATE_RIGHT) { nr = 2 * Dp; nc = 2 * Dn; ncs = nc; }
  else if (st.mode == GATE_LEFT) { nr = 2 * Dn; nc = 2 * Dp; ncs = nc; }
  else if (st.mode == MOVE_RIGHT) { nr = 2 * Dp; nc = Dm; ncs = 2 * Dn; }
  else { nr = 2 * Dn; nc = Dm; ncs = 2 * Dp; }

  // site tensors as matrices: row (s, a) and column c of A_p, row c and
  // column (t, b) of A_{p+1}
  auto ap_at = [&](int y, int c) -> double2 & {
    const int s = phys_of(y, Dp);
    return Ap[(s * Pw + y - s * Dp) * Pm + c];
  };
  auto aq_at = [&](int c, int x) -> double2 & {
    const int t = phys_of(x, Dn);
    return Aq[(t * Pm + c) * Pn + x - t * Dn];
  };

  // ---------------------------------------------------------- build M
  {
    // pair product of the two sites, the two-site tensor before the gate
    // (Fig. 1b): P[(s', a)][(t', b)] = sum_c A_p[s'][a][c] A_{p+1}[t'][c][b]
    double2 pt[ROWS][2];
    staged_tile_gemm<N, W, ROWS>(
        Dm, [&](int y, int c) { return y < 2 * Dp ? ap_at(y, c) : make_double2(0.0, 0.0); },
        [&](int c, int x) { return x < 2 * Dn ? aq_at(c, x) : make_double2(0.0, 0.0); }, sh, pt);
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (row0 + rr < 2 * Dp && c0 + q < 2 * Dn) P2[(row0 + rr) * N + c0 + q] = pt[rr][q];
  }
  step_sync<W>();
  // projection source S[y][x] (y < nr, x < ncs): the gate's theta or its
  // adjoint, which is also the Jacobi matrix, or (centre moves) the pair
  // product or its adjoint
  auto source = [&](int y, int x) {
    const int r = right ? y : x, c = right ? x : y;
    const int s = phys_of(r, Dp), t = phys_of(c, Dn);
    const double2 v = theta_from_pair(P2, gate ? st.op : int(OP_ID), cg, sg, Dp, Dn, s, r - s * Dp, t, c - t * Dn, N);
    return right ? v : cconj(v);
  };
  Columns<N, W> M;
#pragma unroll
  for (int rr = 0; rr < ROWS; ++rr) {
    const int r = row0 + rr;
    double2 v[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = c0 + q;
      v[q] = make_double2(0.0, 0.0);
      if (r < nr && c < nc) {
        if (gate) v[q] = source(r, c);
        else v[q] = right ? ap_at(r, c) : cconj(aq_at(c, r));   // the site being orthogonalised
      }
    }
    M.Ar[rr] = v[0].x;
    M.Ai[rr] = v[0].y;
    M.Br[rr] = v[1].x;
    M.Bi[rr] = v[1].y;
  }
  const double zero_w = lane0(kZeroWeight * row_weights<N, W>(M, sh, nr, tid));   // wave-uniform
  const int nref = min(nr, nc);
  // Up to four columns take fewer sweeps than reflections are worth: of a
  // 20,000-cycle step at bonds up to 2, 5,000 were the LQ and 5,400 the sweeps
  // after it (8 points x 20 qubits, d = 1: 640 -> 555 us without)
  const bool few = N == 16 && nc <= 4;
  if (!few) lq_reduce<N, W>(M, sh, nr, nref, tid);
  const int cols = few ? nc : nref;
  const int NP = max(2, cols + (cols & 1));
  const bool converged = jacobi_sweeps<N, W>(M, sh, NP / 2, zero_w, tid);
  select_columns<N, W>(M, sh, cl, P, st, gate, cg, sg, Dm, nref, NP, zero_w, converged, tid);
  const int k = sh.k;
  const double nrm = sh.nrm;

  // ---------------------------------------------------------- write factors
  // the isometric factor; what the old tensors held beyond column (row) k
  // becomes zero
  auto iso_at = [&](int r, int j) -> double2 & { return right ? ap_at(r, j) : aq_at(j, r); };
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int pos = 2 * cp + q;
    const int j = sh.rank[pos];
    const bool keep = pos < NP && j < k;
    const double inv = keep ? rsqrt(sh.norm[pos]) : 0.0;
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) {
      const int r = row0 + rr;
      if (keep && r < nr) {
        const double vr = (q == 0 ? M.Ar[rr] : M.Br[rr]) * inv;
        const double vi = (q == 0 ? M.Ai[rr] : M.Bi[rr]) * inv;
        iso_at(r, j) = make_double2(vr, right ? vi : -vi);
        if constexpr (Y::kLds) sh.U[r * N + j] = make_double2(vr, vi);
      }
    }
  }
  if (k < Dm) {
    // e / w by reciprocal, exact here: (e + 1/2) / w is at least 1 / (2 w) from any integer
    const int w = Dm - k, w2 = 2 * Dn;
    const float rw = __builtin_amdgcn_rcpf(float(w)), rw2 = __builtin_amdgcn_rcpf(float(w2));
    for (int e = tid; e < 2 * Dp * w; e += Y::T) {
      const int y = int((float(e) + 0.5f) * rw);
      ap_at(y, k + e - y * w) = make_double2(0.0, 0.0);
    }
    for (int e = tid; e < w2 * w; e += Y::T) {
      const int c = int((float(e) + 0.5f) * rw2);
      aq_at(k + c, e - c * w2) = make_double2(0.0, 0.0);
    }
  }
  step_sync<W>();
  // projection: out[j][x] = nrm sum_y conj(U[y][j]) S[y][x] (j < k, x < ncs)
  auto out_at = [&](int j, int x, double2 v) {
    if (right) aq_at(j, x) = make_double2(nrm * v.x, nrm * v.y);
    else ap_at(x, j) = make_double2(nrm * v.x, -nrm * v.y);
  };
  if constexpr (Y::kLds) {
    for (int e = tid; e < k * N; e += Y::T) {
      const int j = e / N, x = e % N;
      if (x < ncs) {
        double2 v = make_double2(0.0, 0.0);
#pragma unroll 4
        for (int y = 0; y < nr; ++y) {
          const double2 u = sh.U[y * N + j], s = source(y, x);
          v.x = fma(u.x, s.x, fma(u.y, s.y, v.x));
          v.y = fma(u.x, s.y, fma(-u.y, s.x, v.y));
        }
        out_at(j, x, v);
      }
    }
  } else {
    // blocks of N / 2 rows j
    for (int j0 = 0; j0 < k; j0 += N / 2) {
      double2 acc[Y::HROWS][2];
      staged_tile_gemm<N, W, Y::HROWS>(
          nr,
          [&](int jj, int y) {
            const int j = j0 + jj;
            if (j >= k) return make_double2(0.0, 0.0);
            const double2 u = iso_at(y, j);
            return right ? cconj(u) : u;
          },
          [&](int y, int x) { return x < ncs ? source(y, x) : make_double2(0.0, 0.0); }, sh, acc);
#pragma unroll
      for (int rr = 0; rr < Y::HROWS; ++rr)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = j0 + (wave * Y::RG + lane / LC) * Y::HROWS + rr, x = c0 + q;
          if (wave < Y::WA && j < k && x < ncs) out_at(j, x, acc[rr][q]);
        }
    }
  }
  if (tid == 0) dims[p + 1] = k;
}

// Two-qubit gate of circuit ci whose Jacobi matrix has more than 128 rows and
// columns (both neighbouring bonds above 64; one 1024-thread workgroup); a
// centre move has at most 128 columns, the cap of its bond.  The same
// operation as svd_step -- pair product, theta, one-sided Jacobi on the
// columns, truncation by Eq. (8) with the bond cap, isometric factor from the
// normalised columns and the other factor as an exact projection -- with the
// matrices in the circuit's global scratch slot (L2-resident) instead of
// registers:
//   W: the pair product (row-major), then the Jacobi matrix M column-major
//      (column c at W + c kWideN, rows 0..255, zero beyond nr);
//   S: the projection source (row-major, row stride kWideN).
// M is first reduced as in svd_step (M <- M H_0 H_1 ..., Householder
// reflections from the right, the heaviest remaining row next), so
// that only its first min(nr, nc) columns carry more than rounding-level
// weight; the Jacobi sweeps then pair those columns, two to a block, in
// round-robin order of the blocks.  Wave w takes block pairs w, w + 16, ... of
// a round with their four columns in registers and rotates the four pairs
// across the blocks (in the first round also the two inside them), so every
// two columns meet once per sweep and a round moves each column through L2
// once for two rotations: single columns made a round of 256 x 256 a transfer
// of 2 MiB at the 125 bytes a cycle that one CU reaches.
// Whole simulation of 4 points x 16 qubits, d = 5, chi 128, whose bonds
// saturate (gates with both bonds above 64 are here, those with one of them in
// svd_step_wide): blocks of two columns 814 -> 664 ms, with the heaviest
// remaining row as the next pivot and the pair product and projection staged
// through LDS 617.  Other points take up to 670: their sweeps differ.
__device__ __attribute__((noinline)) void svd_step_stream(const SvParams *Pq, int64_t ci_, const SimStep *stp, int lds) {
  CircuitLds &cl = *lds_at<CircuitLds>(lds);
  const SvParams P = uniform_load(Pq);
  const SimStep st = uniform_load(stp);
  const int64_t ci = uniform(ci_);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ double w_norm[kWideN];   // squared norm of each Jacobi column (row norms during the LQ)
  __shared__ double w_sorted[kWideN]; // norms in decreasing order
  __shared__ int w_col[kWideN];       // column of each rank
  __shared__ double2 w_vec[kWideN];   // Householder vector of an LQ step
  __shared__ double2 w_dot[4][kWideN];// partial products row . conj(w)
  __shared__ double w_part[kSvWaves];
  __shared__ int w_k;
  __shared__ double w_nrm, w_tot;

  int32_t *dims = P.dims + ci * (P.m + 1);
  const int p = st.p;
  const int Dp = dims[p], Dm = dims[p + 1], Dn = dims[p + 2];
  const int Pp = P.pad[p], Pm = P.pad[p + 1], Pn = P.pad[p + 2];
  double2 *Ap = P.f64 + ci * P.mps_stride + P.site_off[p];
  double2 *Aq = P.f64 + ci * P.mps_stride + P.site_off[p + 1];
  double2 *W = P.wscratch + int64_t(blockIdx.x) * kWideSlot;
  double2 *S = W + kWideN * kWideN;

  double cg = 1.0, sg = 0.0;
  if (st.op == OP_RXX) {
    const double xi = P.X[ci * P.ldx + st.fi], xj = P.X[ci * P.ldx + st.fj];
    const double phi = P.coef_xx * (1.0 - xi) * (1.0 - xj);
    sincos(0.5 * phi, &sg, &cg);
  }
  const bool right = st.mode == GATE_RIGHT;
  const int nr = 2 * (right ? Dp : Dn), nc = 2 * (right ? Dn : Dp);

  // ---------------------------------------------------------- pair product -> W
  // P[(s', a)][(t', b)] = sum_c A_p[s'][a][c] A_{p+1}[t'][c][b]
  using T = Layout<kSvMaxN, kSvWaves>;
  StepLds<kSvMaxN, kSvWaves> &sh = *lds_at<StepLds<kSvMaxN, kSvWaves>>(lds + int(sizeof(CircuitLds)));
  auto ap_at = [&](int y, int c) -> double2 & {
    const int s = phys_of(y, Dp);
    return Ap[(s * Pp + y - s * Dp) * Pm + c];
  };
  auto aq_at = [&](int c, int x) -> double2 & {
    const int t = phys_of(x, Dn);
    return Aq[(t * Pm + c) * Pn + x - t * Dn];
  };
  for (int y0 = 0; y0 < 2 * Dp; y0 += kSvMaxN)
    for (int x0 = 0; x0 < 2 * Dn; x0 += kSvMaxN) {
      double2 pt[T::ROWS][2];
      staged_tile_gemm<kSvMaxN, kSvWaves, T::ROWS>(
          Dm, [&](int y, int c) { return y0 + y < 2 * Dp ? ap_at(y0 + y, c) : make_double2(0.0, 0.0); },
          [&](int c, int x) { return x0 + x < 2 * Dn ? aq_at(c, x0 + x) : make_double2(0.0, 0.0); }, sh, pt);
#pragma unroll
      for (int rr = 0; rr < T::ROWS; ++rr)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int y = y0 + wave * T::ROWS + rr, x = x0 + 2 * lane + q;
          if (y < 2 * Dp && x < 2 * Dn) W[y * kWideN + x] = pt[rr][q];
        }
    }
  __syncthreads();
  // ---------------------------------------------------------- projection source -> S
  // theta (absorb right) or theta^H (absorb left), which is also the Jacobi
  // matrix
  for (int e = tid; e < nr * nc; e += kSvThreads) {
    const int r = e / nc, c = e % nc;
    S[size_t(r) * kWideN + c] =
        right ? theta_from_pair(W, st.op, cg, sg, Dp, Dn, r / Dp, r % Dp, c / Dn, c % Dn, kWideN)
              : cconj(theta_from_pair(W, st.op, cg, sg, Dp, Dn, c / Dp, c % Dp, r / Dn, r % Dn, kWideN));
  }
  __syncthreads();
  // ---------------------------------------------------------- Jacobi matrix -> W (column-major)
  // with ||M||_F^2 (invariant under the rotations)
  {
    double t = 0.0;
    for (int e = tid; e < nc * kWideN; e += kSvThreads) {
      const int c = e / kWideN, r = e % kWideN;
      const double2 v = r < nr ? S[size_t(r) * kWideN + c] : make_double2(0.0, 0.0);
      W[size_t(c) * kWideN + r] = v;
      t = fma(v.x, v.x, fma(v.y, v.y, t));
    }
    t = wave_sum(t);
    if (lane == 0) w_part[wave] = t;
    __syncthreads();
    if (tid == 0) {
      double u = 0.0;
      for (int w = 0; w < kSvWaves; ++w) u += w_part[w];
      w_tot = u;
    }
    __syncthreads();
  }
  const double zero_w = lane0(kZeroWeight * w_tot);

  // ---------------------------------------------------------- LQ preconditioning
  // Step i reflects the heaviest remaining row x (restricted to columns >= i)
  // onto column i: w = x + e^{i arg x_i} |x| e_i, beta = 1 / (|x| (|x| + |x_i|)),
  // every row r <- r - beta (r . conj w) w.  Thread (r, q) = (tid % 256,
  // tid / 256) takes row r and the columns c = i + q mod 4, the first of them
  // held in registers between the product and the update.
  const int nref = min(nr, nc);
  {
    if (tid < kWideN) {
      double t = 0.0;
      if (tid < nr)
        for (int c = 0; c < nc; ++c) {
          const double2 v = W[size_t(c) * kWideN + tid];
          t = fma(v.x, v.x, fma(v.y, v.y, t));
        }
      w_norm[tid] = tid < nr ? t : -1.0;
    }
    __syncthreads();
    const int r = tid & (kWideN - 1), q = tid >> 8;
    for (int i = 0; i < nref; ++i) {
      const int pv = __builtin_amdgcn_readfirstlane(heaviest_row<kWideN>(w_norm, lane));
      if (tid < kWideN) {
        // the pivot row restricted to columns >= i, and |x|
        const double2 x = (tid >= i && tid < nc) ? W[size_t(tid) * kWideN + pv] : make_double2(0.0, 0.0);
        w_vec[tid] = x;
        const double n2 = wave_sum(fma(x.x, x.x, x.y * x.y));
        if (lane == 0) w_part[wave] = n2;
      }
      __syncthreads();
      const double n2 = (w_part[0] + w_part[1]) + (w_part[2] + w_part[3]);
      const double2 xi = w_vec[i];
      const double a2 = fma(xi.x, xi.x, xi.y * xi.y);
      const double rx = n2 > 0.0 ? rsqrt(n2) : 0.0, ra = a2 > 0.0 ? rsqrt(a2) : 0.0;
      const double nx = n2 * rx, ax = a2 * ra;
      const double2 wi = make_double2((a2 > 0.0 ? xi.x * ra : 1.0) * (ax + nx), xi.y * ra * (ax + nx));
      const double beta = n2 > 0.0 ? rx * reciprocal(nx + ax) : 0.0;
      constexpr int kHeld = 12;
      double2 held[kHeld];
      double dr = 0.0, di = 0.0;
      auto add = [&](const double2 &v, const double2 &w) {
        dr = fma(v.x, w.x, fma(v.y, w.y, dr));
        di = fma(v.y, w.x, fma(-v.x, w.y, di));
      };
      double2 *mine = W + r;
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        const int c = i + q + 4 * u;
        held[u] = c < nc && r < nr ? mine[c * kWideN] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        const int c = i + q + 4 * u;
        if (c < nc) add(held[u], c == i ? wi : w_vec[c]);
      }
      if (r < nr)
        for (int c = i + q + 4 * kHeld; c < nc; c += 4) add(mine[c * kWideN], w_vec[c]);
      w_dot[q][r] = make_double2(dr, di);
      __syncthreads();
      if (r < nr) {
        const double2 d0 = w_dot[0][r], d1 = w_dot[1][r], d2 = w_dot[2][r], d3 = w_dot[3][r];
        dr = beta * ((d0.x + d1.x) + (d2.x + d3.x));
        di = beta * ((d0.y + d1.y) + (d2.y + d3.y));
        auto less = [&](const double2 &v, const double2 &w) {
          return make_double2(v.x - (dr * w.x - di * w.y), v.y - (dr * w.y + di * w.x));
        };
#pragma unroll
        for (int u = 0; u < kHeld; ++u) {
          const int c = i + q + 4 * u;
          if (c < nc) {
            const double2 v = less(held[u], c == i ? wi : w_vec[c]);
            mine[c * kWideN] = v;
            if (c == i) {
              const double w = w_norm[r];
              w_norm[r] = r == pv || w < 0.0 ? -1.0 : fmax(w - fma(v.x, v.x, v.y * v.y), 0.0);
            }
          }
        }
        for (int c = i + q + 4 * kHeld; c < nc; c += 4) mine[c * kWideN] = less(mine[c * kWideN], w_vec[c]);
      }
      __syncthreads();  // the next step reads its pivot row and rewrites the LDS vectors
    }
  }

  // ---------------------------------------------------------- Jacobi sweeps
  const int NP = max(2, nref + (nref & 1));
  bool converged = false;
  // columns in blocks of two (an even number of them, the last perhaps empty)
  const int blocks = NP / 2, even = blocks + (blocks & 1), rounds = even - 1;
  using Column = double2[4];   // rows lane + 64 q
  for (int sweep = 0; sweep < kMaxSweeps && !converged; ++sweep) {
    bool large = false;
    for (int rd = 0; rd < rounds; ++rd) {
      for (int k = wave; k < even / 2; k += kSvWaves) {
        // round-robin pairing: the last block meets block rd, the others pair
        // symmetrically around rd (indices mod even - 1)
        const int i = k == 0 ? even - 1 : (rd + k) % rounds;
        const int j = k == 0 ? rd : (rd - k + rounds) % rounds;
        Column x[2], y[2];
        double w[4] = {0.0, 0.0, 0.0, 0.0};   // squared norms of x, y
        double2 *X = W + size_t(2 * i) * kWideN + lane, *Y = W + size_t(2 * j) * kWideN + lane;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            x[c][q] = i < blocks ? X[c * kWideN + 64 * q] : make_double2(0.0, 0.0);
            y[c][q] = j < blocks ? Y[c * kWideN + 64 * q] : make_double2(0.0, 0.0);
          }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            w[c] = fma(x[c][q].x, x[c][q].x, fma(x[c][q].y, x[c][q].y, w[c]));
            w[2 + c] = fma(y[c][q].x, y[c][q].x, fma(y[c][q].y, y[c][q].y, w[2 + c]));
          }
        wave_sum4(w);
        bool moved = false;
        auto rotate = [&](Column &u, Column &v, double &nu, double &nv, double gr, double gi) {
          const double g2 = fma(gr, gr, gi * gi);
          if (nu > zero_w && nv > zero_w && g2 > (kJacobiTol * kJacobiTol) * (nu * nv)) {
            if (g2 > (kJacobiLarge * kJacobiLarge) * (nu * nv)) large = true;
            moved = true;
            const Rotation r = rotation(nu, nv, gr, gi, g2);
            nu = fmax(nu - r.tg, 0.0);
            nv += r.tg;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const double2 a = u[q], b = v[q];
              u[q] = make_double2(fma(r.c, a.x, fma(-r.sr, b.x, r.si * b.y)), fma(r.c, a.y, fma(-r.sr, b.y, -r.si * b.x)));
              v[q] = make_double2(fma(r.c, b.x, fma(r.sr, a.x, r.si * a.y)), fma(r.c, b.y, fma(r.sr, a.y, -r.si * a.x)));
            }
          }
        };
        // two disjoint pairs at once
        auto rotate2 = [&](Column &u0, Column &v0, double &nu0, double &nv0, Column &u1, Column &v1, double &nu1,
                           double &nv1) {
          double g[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            g[0] = fma(u0[q].x, v0[q].x, fma(u0[q].y, v0[q].y, g[0]));
            g[1] = fma(u0[q].x, v0[q].y, fma(-u0[q].y, v0[q].x, g[1]));
            g[2] = fma(u1[q].x, v1[q].x, fma(u1[q].y, v1[q].y, g[2]));
            g[3] = fma(u1[q].x, v1[q].y, fma(-u1[q].y, v1[q].x, g[3]));
          }
          wave_sum4(g);
          rotate(u0, v0, nu0, nv0, g[0], g[1]);
          rotate(u1, v1, nu1, nv1, g[2], g[3]);
        };
        if (rd == 0) rotate2(x[0], x[1], w[0], w[1], y[0], y[1], w[2], w[3]);   // inside the blocks
        rotate2(x[0], y[0], w[0], w[2], x[1], y[1], w[1], w[3]);
        rotate2(x[0], y[1], w[0], w[3], x[1], y[0], w[1], w[2]);
        if (moved) {
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if (i < blocks) X[c * kWideN + 64 * q] = x[c][q];
              if (j < blocks) Y[c * kWideN + 64 * q] = y[c][q];
            }
        }
      }
      __syncthreads();  // the next round reads the columns this one wrote
    }
    converged = __syncthreads_or(large ? 1 : 0) == 0;
  }

  // ---------------------------------------------------------- norms, order, k
  for (int c = wave; c < kWideN; c += kSvWaves) {
    double t = 0.0;
    if (c < NP) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double2 v = W[size_t(c) * kWideN + lane + 64 * q];
        t = fma(v.x, v.x, fma(v.y, v.y, t));
      }
      t = wave_sum(t);
    }
    if (lane == 0) w_norm[c] = t;
  }
  __syncthreads();
  if (tid < kWideN) {
    const double v = w_norm[tid];
    int rank = 0;
#pragma unroll 1
    for (int u = 0; u < kWideN; ++u) {
      const double o = w_norm[u];
      rank += (o > v || (o == v && u < tid)) ? 1 : 0;
    }
    w_sorted[rank] = v;
    w_col[rank] = tid;
  }
  __syncthreads();
  if (tid == 0) {
    const int nsv = min(nr, nc);
    int nnz = 0;
#pragma unroll 1
    for (int u = 0; u < kWideN; ++u) nnz += w_sorted[u] > zero_w ? 1 : 0;
    double total = 0.0;
#pragma unroll 1
    for (int u = kWideN - 1; u >= 0; --u) total += w_sorted[u];
    int kcut = nsv;
    if (P.cutoff > 0.0) {
      // smallest k with sum_{r >= k} w_r <= cutoff * total
      double tail = 0.0;
#pragma unroll 1
      for (int kk = nsv; kk >= 0; --kk) {
        if (kk < nsv) tail += w_sorted[kk];
        if (tail <= P.cutoff * total) kcut = kk;
        else break;
      }
    }
    int k = max(1, min(min(P.chi, kcut), max(nnz, 1)));
    if (P.gate_split) {
      const double cmax = fmax(fabs(cg), fabs(sg));
      const int rg = st.op == OP_RXX ? (fabs(cg) > 1e-12 * cmax ? 1 : 0) + (fabs(sg) > 1e-12 * cmax ? 1 : 0) : 4;
      k = max(1, min(k, rg * Dm));
    }
    k = min(k, st.nr);
    double kept = 0.0;
#pragma unroll 1
    for (int u = k - 1; u >= 0; --u) kept += w_sorted[u];
    double tail = 0.0;
#pragma unroll 1
    for (int u = kWideN - 1; u >= k; --u) tail += w_sorted[u];
    const double disc = total > 0.0 ? tail / total : 0.0;
    w_nrm = kept > 0.0 ? 1.0 / sqrt(kept) : 1.0;
    cl.disc += disc;
    cl.maxdisc = fmax(cl.maxdisc, disc);
    if (k < nsv && w_sorted[0] > 0.0 &&
        (sqrt(w_sorted[k - 1]) - sqrt(w_sorted[k])) / sqrt(w_sorted[0]) < kDegenerateGap)
      cl.degen += 1;
    if (!converged) cl.unconv += 1;
    w_k = k;
  }
  __syncthreads();
  const int k = w_k;
  const double nrm = w_nrm;

  // ---------------------------------------------------------- write factors
  for (int e = tid; e < 2 * Pp * Pm; e += kSvThreads) Ap[e] = make_double2(0.0, 0.0);
  for (int e = tid; e < 2 * Pm * Pn; e += kSvThreads) Aq[e] = make_double2(0.0, 0.0);
  __syncthreads();
  // isometric factor: U[:, j] = column w_col[j] / its norm
  for (int e = tid; e < k * nr; e += kSvThreads) {
    const int j = e / nr, r = e % nr;
    const int c = w_col[j];
    const double inv = 1.0 / sqrt(w_norm[c]);
    const double2 v = W[size_t(c) * kWideN + r];
    const double vr = v.x * inv, vi = v.y * inv;
    if (right) Ap[(size_t(r / Dp) * Pp + r % Dp) * Pm + j] = make_double2(vr, vi);
    else Aq[(size_t(r / Dn) * Pm + j) * Pn + r % Dn] = make_double2(vr, -vi);
  }
  // projection: out[j][x] = nrm sum_y conj(U[y][j]) S[y][x]
  for (int x0 = 0; x0 < nc; x0 += kSvMaxN)
    for (int j0 = 0; j0 < k; j0 += kSvMaxN / 2) {
      double2 acc[T::HROWS][2];
      staged_tile_gemm<kSvMaxN, kSvWaves, T::HROWS>(
          nr,
          [&](int jj, int y) {
            if (j0 + jj >= k) return make_double2(0.0, 0.0);
            const int c = w_col[j0 + jj];
            const double inv = rsqrt(w_norm[c]);
            const double2 u = W[c * kWideN + y];
            return make_double2(inv * u.x, -inv * u.y);
          },
          [&](int y, int x) { return x0 + x < nc ? S[y * kWideN + x0 + x] : make_double2(0.0, 0.0); }, sh, acc);
#pragma unroll
      for (int rr = 0; rr < T::HROWS; ++rr)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = j0 + wave * T::HROWS + rr, x = x0 + 2 * lane + q;
          const double2 v = acc[rr][q];
          if (j < k && x < nc) {
            if (right) aq_at(j, x) = make_double2(nrm * v.x, nrm * v.y);
            else ap_at(x, j) = make_double2(nrm * v.x, -nrm * v.y);
          }
        }
    }
  if (tid == 0) dims[p + 1] = k;
}

// Two-site step of circuit ci next to a bond above 64 whose Jacobi matrix M
// (nr x nc, up to 256 either way) has at most 128 rows or at most 128
// columns (one 1024-thread workgroup).  The shorter side fits the registers
// of svd_step once the longer one is reduced, in the circuit's global scratch
// slot (L2-resident): with B = M (wide) or M^H (tall) of at most 128 rows,
//   B H_0 H_1 ... = L  (Householder reflections from the right as in
// lq_reduce), of which only the first columns are not zero.  A wide M has the
// singular vectors of L.  A tall M is H_0 H_1 ... L^H: the columns of L^H go
// through lq_reduce and the sweeps, and the reflections, in reverse, turn
// their orthogonal columns into those of M.
// Scratch slot: B column-major (column c at W + c kWideN), the pair product
// (row-major, kWideN), and the reflection vectors of a tall M with their
// factors.
// With the sweeps streaming the columns from L2 instead (every round of 256 x
// 128 columns ~7 us): 594 ms against 270 for 4 points x 16 qubits, d = 5, chi
// 128, on points whose bonds stay below the cap, so that nearly every step next
// to a bond above 64 has one side within 128.
struct WideLds {
  double2 vec[kWideN];          // pivot row of a reflection
  double2 dot[8][kSvMaxN];      // partial products row . conj(w)
  double rn[kSvMaxN];           // remaining row norms
  double part[kSvWaves];
};

__device__ __attribute__((noinline)) void svd_step_wide(const SvParams *Pq, int64_t ci_, const SimStep *stp, int lds,
                                                        int Dp_, int Dm_, int Dn_) {
  constexpr int N = kSvMaxN, W = kSvWaves;
  using Y = Layout<N, W>;
  constexpr int ROWS = Y::ROWS;
  CircuitLds &cl = *lds_at<CircuitLds>(lds);
  StepLds<N, W> &sh = *lds_at<StepLds<N, W>>(lds + int(sizeof(CircuitLds)));
  static_assert(sizeof(WideLds) <= sizeof(sh.stage), "the reflection buffers lie over the staging buffers");
  WideLds &wl = *reinterpret_cast<WideLds *>(&sh.stage);
  const SvParams P = uniform_load(Pq);
  const SimStep st = uniform_load(stp);
  const int64_t ci = uniform(ci_);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  int32_t *dims = P.dims + ci * (P.m + 1);
  const int p = st.p;
  const int Dp = uniform(Dp_), Dm = uniform(Dm_), Dn = uniform(Dn_);
  const int Pw = st.Pp, Pm = st.Pm, Pn = st.Pn;
  double2 *Ap = P.f64 + ci * P.mps_stride + st.off_p;
  double2 *Aq = P.f64 + ci * P.mps_stride + st.off_q;
  double2 *B = P.wscratch + int64_t(blockIdx.x) * kWideSlot;
  double2 *P2 = B + kWideN * kWideN;
  double2 *V = P2 + kWideN * kWideN;                                   // reflection i at V + i kWideN
  double *betas = reinterpret_cast<double *>(V + kSvMaxN * kWideN);

  double cg = 1.0, sg = 0.0;
  if (st.op == OP_RXX) {
    const double xi = P.X[ci * P.ldx + st.fi], xj = P.X[ci * P.ldx + st.fj];
    const double phi = P.coef_xx * (1.0 - xi) * (1.0 - xj);
    sincos(0.5 * phi, &sg, &cg);
  }
  const bool right = (st.mode == GATE_RIGHT || st.mode == MOVE_RIGHT);
  const bool gate = (st.mode == GATE_RIGHT || st.mode == GATE_LEFT);
  int nr, nc, ncs;
  if (st.mode == GATE_RIGHT) { nr = 2 * Dp; nc = 2 * Dn; ncs = nc; }
  else if (st.mode == GATE_LEFT) { nr = 2 * Dn; nc = 2 * Dp; ncs = nc; }
  else if (st.mode == MOVE_RIGHT) { nr = 2 * Dp; nc = Dm; ncs = 2 * Dn; }
  else { nr = 2 * Dn; nc = Dm; ncs = 2 * Dp; }
  auto ap_at = [&](int y, int c) -> double2 & {
    const int s = phys_of(y, Dp);
    return Ap[(s * Pw + y - s * Dp) * Pm + c];
  };
  auto aq_at = [&](int c, int x) -> double2 & {
    const int t = phys_of(x, Dn);
    return Aq[(t * Pm + c) * Pn + x - t * Dn];
  };

  // ---------------------------------------------------------- pair product
  for (int y0 = 0; y0 < 2 * Dp; y0 += N)
    for (int x0 = 0; x0 < 2 * Dn; x0 += N) {
      double2 pt[ROWS][2];
      staged_tile_gemm<N, W, ROWS>(
          Dm, [&](int y, int c) { return y0 + y < 2 * Dp ? ap_at(y0 + y, c) : make_double2(0.0, 0.0); },
          [&](int c, int x) { return x0 + x < 2 * Dn ? aq_at(c, x0 + x) : make_double2(0.0, 0.0); }, sh, pt);
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int y = y0 + wave * ROWS + rr, x = x0 + 2 * lane + q;
          if (y < 2 * Dp && x < 2 * Dn) P2[y * kWideN + x] = pt[rr][q];
        }
    }
  __syncthreads();
  auto source = [&](int y, int x) {
    const int r = right ? y : x, c = right ? x : y;
    const int s = phys_of(r, Dp), t = phys_of(c, Dn);
    const double2 v =
        theta_from_pair(P2, gate ? st.op : int(OP_ID), cg, sg, Dp, Dn, s, r - s * Dp, t, c - t * Dn, kWideN);
    return right ? v : cconj(v);
  };
  auto matrix = [&](int r, int c) {   // M
    return gate ? source(r, c) : right ? ap_at(r, c) : cconj(aq_at(c, r));
  };

  // ---------------------------------------------------------- the longer side
  const bool tall = nr > N;
  const int rb = tall ? nc : nr, cb = tall ? nr : nc;   // B: rb <= 128 rows
  if (cb > N) {
    const int r = tid & (N - 1), q = tid >> 7;   // row and columns q, q + 8, ... of this thread
    double w2 = 0.0;
    for (int c = q; c < cb; c += 8) {
      double2 v = make_double2(0.0, 0.0);
      if (r < rb) v = tall ? cconj(matrix(c, r)) : matrix(r, c);
      B[c * kWideN + r] = v;
      w2 = fma(v.x, v.x, fma(v.y, v.y, w2));
    }
    wl.dot[q][r] = make_double2(w2, 0.0);
    __syncthreads();
    if (tid < N) {
      double t = 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) t += wl.dot[u][tid].x;
      wl.rn[tid] = tid < rb ? t : -1.0;
    }
    __syncthreads();
    for (int i = 0; i < rb; ++i) {
      const int pv = __builtin_amdgcn_readfirstlane(heaviest_row<N>(wl.rn, lane));
      if (tid < kWideN) {
        const double2 x = (tid >= i && tid < cb) ? B[tid * kWideN + pv] : make_double2(0.0, 0.0);
        wl.vec[tid] = x;
        const double n2 = wave_sum(fma(x.x, x.x, x.y * x.y));
        if (lane == 0) wl.part[wave] = n2;
      }
      __syncthreads();
      const double n2 = (wl.part[0] + wl.part[1]) + (wl.part[2] + wl.part[3]);
      const double2 xi = wl.vec[i];
      const double a2 = fma(xi.x, xi.x, xi.y * xi.y);
      const double rx = n2 > 0.0 ? rsqrt(n2) : 0.0, ra = a2 > 0.0 ? rsqrt(a2) : 0.0;
      const double nx = n2 * rx, ax = a2 * ra;
      const double2 wi = make_double2((a2 > 0.0 ? xi.x * ra : 1.0) * (ax + nx), xi.y * ra * (ax + nx));
      const double beta = n2 > 0.0 ? rx * reciprocal(nx + ax) : 0.0;
      if (tall) {
        if (tid < kWideN) V[i * kWideN + tid] = tid == i ? wi : wl.vec[tid];
        if (tid == 0) betas[i] = beta;
      }
      // this thread's columns from i on; the first 12 of them stay in registers
      constexpr int kHeld = 12;
      const int cf = i + ((q - i) & 7);
      double2 held[kHeld];
      double dr = 0.0, di = 0.0;
      auto add = [&](const double2 &v, const double2 &w) {
        dr = fma(v.x, w.x, fma(v.y, w.y, dr));
        di = fma(v.y, w.x, fma(-v.x, w.y, di));
      };
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        const int c = cf + 8 * u;
        held[u] = c < cb ? B[c * kWideN + r] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        const int c = cf + 8 * u;
        if (c < cb) add(held[u], c == i ? wi : wl.vec[c]);
      }
      for (int c = cf + 8 * kHeld; c < cb; c += 8) add(B[c * kWideN + r], wl.vec[c]);
      wl.dot[q][r] = make_double2(dr, di);
      __syncthreads();
      dr = di = 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const double2 v = wl.dot[u][r];
        dr += v.x;
        di += v.y;
      }
      dr *= beta;
      di *= beta;
      auto less = [&](const double2 &v, const double2 &w) {
        return make_double2(v.x - (dr * w.x - di * w.y), v.y - (dr * w.y + di * w.x));
      };
#pragma unroll
      for (int u = 0; u < kHeld; ++u) {
        const int c = cf + 8 * u;
        if (c < cb) {
          const double2 v = less(held[u], c == i ? wi : wl.vec[c]);
          B[c * kWideN + r] = v;
          if (c == i && r < rb) {
            const double w = wl.rn[r];
            wl.rn[r] = r == pv || w < 0.0 ? -1.0 : fmax(w - fma(v.x, v.x, v.y * v.y), 0.0);
          }
        }
      }
      for (int c = cf + 8 * kHeld; c < cb; c += 8) {
        double2 *m = B + c * kWideN + r;
        *m = less(*m, wl.vec[c]);
      }
      __syncthreads();   // the next pivot row is complete
    }
  }

  // ---------------------------------------------------------- sweeps in registers
  const int row0 = wave * ROWS, c0 = 2 * lane;
  const int nref = min(nr, nc);
  Columns<N, W> M;
#pragma unroll
  for (int rr = 0; rr < ROWS; ++rr) {
    const int r = row0 + rr;
    double2 v[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = c0 + q;
      v[q] = make_double2(0.0, 0.0);
      if (cb <= N) {
        if (r < nr && c < nc) v[q] = matrix(r, c);
      } else if (r < nref && c < nref) {
        v[q] = tall ? cconj(B[r * kWideN + c]) : B[c * kWideN + r];
      }
    }
    M.Ar[rr] = v[0].x;
    M.Ai[rr] = v[0].y;
    M.Br[rr] = v[1].x;
    M.Bi[rr] = v[1].y;
  }
  __syncthreads();   // the reflection buffers are free
  const int rows = tall ? nref : nr;
  const double zero_w = lane0(kZeroWeight * row_weights<N, W>(M, sh, rows, tid));   // wave-uniform
  if (tall || cb <= N) lq_reduce<N, W>(M, sh, rows, nref, tid);   // (a wide M is L already)
  const int NP = max(2, nref + (nref & 1));
  const bool converged = jacobi_sweeps<N, W>(M, sh, NP / 2, zero_w, tid);
  select_columns<N, W>(M, sh, cl, P, st, gate, cg, sg, Dm, nref, NP, zero_w, converged, tid);
  const int k = sh.k;
  const double nrm = sh.nrm;

  // ---------------------------------------------------------- write factors
  auto iso_at = [&](int r, int j) -> double2 & { return right ? ap_at(r, j) : aq_at(j, r); };
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int pos = c0 + q;
    const int j = sh.rank[pos];
    const bool keep = pos < NP && j < k;
    const double inv = keep ? rsqrt(sh.norm[pos]) : 0.0;
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) {
      const int r = row0 + rr;
      if (keep && r < rows) {
        const double vr = (q == 0 ? M.Ar[rr] : M.Br[rr]) * inv;
        const double vi = (q == 0 ? M.Ai[rr] : M.Bi[rr]) * inv;
        if (tall) B[j * kWideN + r] = make_double2(vr, vi);
        else iso_at(r, j) = make_double2(vr, right ? vi : -vi);
      }
    }
  }
  if (tall) {
    __syncthreads();
    // column j <- H_0 ... H_{nref-1} (column, 0): 32 lanes per column, lane hl
    // rows hl + 32 q
    const int hl = lane & 31;
    for (int j = 2 * wave + (lane >> 5); j < k + (k & 1); j += 2 * W) {
      double2 u[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = hl + 32 * q;
        u[q] = r < nref && j < k ? B[j * kWideN + r] : make_double2(0.0, 0.0);
      }
      for (int i = nref - 1; i >= 0; --i) {
        const double beta = betas[i];
        double2 w[8];
        double dr = 0.0, di = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) w[q] = V[i * kWideN + hl + 32 * q];
#pragma unroll
        for (int q = 0; q < 8; ++q) {   // H = 1 - beta conj(w) w^T
          dr = fma(w[q].x, u[q].x, fma(-w[q].y, u[q].y, dr));
          di = fma(w[q].x, u[q].y, fma(w[q].y, u[q].x, di));
        }
        dr = beta * cols_sum<32>(dr);
        di = beta * cols_sum<32>(di);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          u[q].x -= w[q].x * dr + w[q].y * di;
          u[q].y -= w[q].x * di - w[q].y * dr;
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = hl + 32 * q;
        if (j < k && r < nr) iso_at(r, j) = make_double2(u[q].x, right ? u[q].y : -u[q].y);
      }
    }
  }
  if (k < Dm) {
    // e / w by reciprocal, exact here: (e + 1/2) / w is at least 1 / (2 w) from any integer
    const int w = Dm - k, w2 = 2 * Dn;
    const float rw = __builtin_amdgcn_rcpf(float(w)), rw2 = __builtin_amdgcn_rcpf(float(w2));
    for (int e = tid; e < 2 * Dp * w; e += Y::T) {
      const int y = int((float(e) + 0.5f) * rw);
      ap_at(y, k + e - y * w) = make_double2(0.0, 0.0);
    }
    for (int e = tid; e < w2 * w; e += Y::T) {
      const int c = int((float(e) + 0.5f) * rw2);
      aq_at(k + c, e - c * w2) = make_double2(0.0, 0.0);
    }
  }
  __syncthreads();
  // projection: out[j][x] = nrm sum_y conj(U[y][j]) S[y][x] (j < k, x < ncs)
  for (int x0 = 0; x0 < ncs; x0 += N)
    for (int j0 = 0; j0 < k; j0 += N / 2) {
      double2 acc[Y::HROWS][2];
      staged_tile_gemm<N, W, Y::HROWS>(
          nr,
          [&](int jj, int y) {
            const int j = j0 + jj;
            if (j >= k) return make_double2(0.0, 0.0);
            const double2 u = iso_at(y, j);
            return right ? cconj(u) : u;
          },
          [&](int y, int x) { return x0 + x < ncs ? source(y, x0 + x) : make_double2(0.0, 0.0); }, sh, acc);
#pragma unroll
      for (int rr = 0; rr < Y::HROWS; ++rr)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int j = j0 + wave * Y::HROWS + rr, x = x0 + c0 + q;
          const double2 v = acc[rr][q];
          if (j < k && x < ncs) {
            if (right) aq_at(j, x) = make_double2(nrm * v.x, nrm * v.y);
            else ap_at(x, j) = make_double2(nrm * v.x, -nrm * v.y);
          }
        }
    }
  if (tid == 0) dims[p + 1] = k;
}

// Rz on a run of gate records (Fig. 1a) for circuit ci: A[site][s] *=
// exp(-/+ i theta / 2), one record per wave.  The records of a run act on
// distinct sites, but for circuits without two-qubit gates, whose layers are
// one run: their bonds are 1, so one wave takes the records in order.
template <int W>
__device__ inline void rz_run(const SvParams &P, int64_t ci, const qk_gate *recs, int n_recs, double coef_z) {
  const int lane = threadIdx.x & 63;
  for (int r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); r < n_recs; r += W) {
    const qk_gate g = recs[r];
    const double th = coef_z * P.X[ci * P.ldx + g.feat_i];
    double sn, cs;
    sincos(0.5 * th, &sn, &cs);
    const int32_t *dims = P.dims + ci * (P.m + 1) + g.site;
    const int dl = dims[0], dr = dims[1], pl = P.pad[g.site], pr = P.pad[g.site + 1];
    double2 *A = P.f64 + ci * P.mps_stride + P.site_off[g.site];
    for (int e = lane; e < 2 * dl * dr; e += 64) {
      const int y = e / dr, s = phys_of(y, dl);
      double2 *x = A + (s * pl + y - s * dl) * pr + e % dr;
      const double2 v = *x;
      const double ph = s ? sn : -sn;  // s = 0: exp(-i th/2), s = 1: exp(+i th/2)
      *x = make_double2(cs * v.x - ph * v.y, cs * v.y + ph * v.x);
    }
  }
}

// Steps [s0, s1) of the step list for every circuit, one workgroup each.
// Circuits do not wait for one another between steps, so a launch lasts as
// long as the slowest circuit's total over the chunk rather than the sum,
// over the steps, of each step's slowest SVD (whose sweep count varies from
// circuit to circuit).  NK: the largest Jacobi matrix that the circuit's
// bonds allow; every step takes the smallest kernel that holds its own.  The
// rounds of a sweep are bound by the latency of their reduction, rotation
// and barriers until the matrix nears 128 x 128 (there by the FP64 VALU), so
// what counts is fewer lanes on empty rows, fewer waves to wait for, and
// several circuits per CU: NK = 16 takes one wave per circuit, 32 four (two:
// 9.6 -> 11.3 ms for 128 x 50, d = 2), 64 four with 256 registers per lane
// (eight with 128 take the same alone, but every wave forms the rotations of
// a round, and two circuits on a CU then share its issue slots: 300 x 60,
// d = 3: 168 -> 147 ms; 300 x 40 103.6 -> 90.8), 128 sixteen (eight with 256
// registers gain nothing on 16 x 18, d = 8, and lose a tenth next to bonds
// above 64).  Against one 128 x 128 kernel of 16 waves for every step: 8 points
// x 20 qubits, d = 1: 5.5 -> 0.54 ms; 512 x 165, d = 1: 112 -> 3.5 ms; 128 x 50,
// d = 2: 82 -> 9.0 ms; 300 x 60, d = 3 (two circuits per CU on 44 of 256 CUs):
// 885 -> 143 ms; 16 x 18, d = 8 (saturated at 64): 663 -> 325 ms.
constexpr int sim_waves(int nk) { return nk == 16 ? 1 : nk == 32 ? 4 : nk == 64 ? 4 : 16; }

template <int NK>
constexpr size_t sim_lds_bytes() {
  constexpr int W = sim_waves(NK);
  size_t b = sizeof(StepLds<16, 1>);
  if constexpr (NK >= 32) b = std::max(b, sizeof(StepLds<32, W>));
  if constexpr (NK >= 64) b = std::max(b, sizeof(StepLds<64, W>));
  if constexpr (NK >= 128) b = std::max(b, sizeof(StepLds<128, W>));
  return sizeof(CircuitLds) + b;
}

template <int NK>
__global__ __launch_bounds__(64 * sim_waves(NK), NK == 64 ? 2 : 4) void sim_steps_kernel(const SvParams *Pp,
                                                                          const SimStep *steps, int s0, int s1,
                                                                          const qk_gate *recs, double coef_z) {
  constexpr int W = sim_waves(NK);
  extern __shared__ __align__(16) uint8_t lds_bytes[];
  // The LDS address is handed to the steps as a number that the compiler
  // cannot trace: as a pointer it is taken for the same everywhere, and the
  // steps (shared by several kernels) fetch it from a table in global memory
  // again and again, in every Jacobi round.
  int lds = int(uint32_t(uintptr_t((LdsBytes *)lds_bytes)));
  asm volatile("" : "+s"(lds));
  const SvParams P = uniform_load(Pp);
  const int64_t ci = uniform(circuit_of(P.base));
  if (ci >= P.n) return;
  CircuitLds &cl = *lds_at<CircuitLds>(lds);   // read and written by thread 0 alone
  if (threadIdx.x == 0) cl = CircuitLds{P.disc[ci], P.maxdisc[ci], P.degen[ci], P.unconv[ci], 0};
  for (int s = s0; s < s1; ++s) {
    const SimStep *stp = steps + s;
    const SimStep st = uniform_load(stp);
    if (st.kind == STEP_RZ) {
      rz_run<W>(P, ci, recs + st.r0, st.nr, coef_z);
    } else {
      const int32_t *dims = P.dims + ci * (P.m + 1) + st.p;
      const int Dp = uniform(dims[0]), Dm = uniform(dims[1]), Dn = uniform(dims[2]);
      // every wave has read the bonds, by which it takes its kernel, before
      // one (a step of one wave) rewrites them
      if constexpr (NK > 16) __syncthreads();
      // rows and columns of the Jacobi matrix and of the projection source
      int size = 2 * max(Dp, Dn);
      if (st.mode == MOVE_RIGHT || st.mode == MOVE_LEFT) size = max(size, Dm);
      if constexpr (NK == 16) {
        svd_step<16, 1>(Pp, ci, stp, lds, Dp, Dm, Dn);
      } else {
        if (size <= 16) {
          if (threadIdx.x < 64) svd_step<16, 1>(Pp, ci, stp, lds, Dp, Dm, Dn);
        } else if (NK == 32 || size <= 32) {
          svd_step<32, W>(Pp, ci, stp, lds, Dp, Dm, Dn);
        } else {
          if constexpr (NK >= 64) {
            if (NK == 64 || size <= 64) {
              svd_step<64, W>(Pp, ci, stp, lds, Dp, Dm, Dn);
            } else {
              if constexpr (NK >= 128) {
                if (P.wscratch && (Dp > kWideFrom || Dn > kWideFrom)) {
                  // rows and columns of the Jacobi matrix
                  const int rows = 2 * (st.mode == GATE_RIGHT || st.mode == MOVE_RIGHT ? Dp : Dn);
                  const int cols = st.mode == GATE_RIGHT ? 2 * Dn : st.mode == GATE_LEFT ? 2 * Dp : Dm;
                  if (min(rows, cols) <= kSvMaxN) svd_step_wide(Pp, ci, stp, lds, Dp, Dm, Dn);
                  else svd_step_stream(Pp, ci, stp, lds);
                } else {
                  svd_step<128, W>(Pp, ci, stp, lds, Dp, Dm, Dn);
                }
              }
            }
          }
        }
      }
    }
    step_sync<W>();  // the next step reads the tensors and bond dims this one wrote
    if (P.trace && st.kind == STEP_TWO_SITE && st.r0 >= 0 && threadIdx.x < 64) {
      // memory trace after a two-qubit gate: the bond at its cut and
      // sum_l D_l D_{l+1} (complex entries per physical index) over the MPS.
      // Only reads of the bond dims, which the next step's first thread
      // rewrites after this wave has passed here.
      const int32_t *dims = P.dims + ci * (P.m + 1);
      int acc = 0;
      for (int l = threadIdx.x; l < P.m; l += 64) acc += dims[l] * dims[l + 1];
      for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
      if (threadIdx.x == 0) {
        int32_t *t = P.trace + (ci * P.trace_n2q + st.r0) * 2;
        t[0] = dims[st.p + 1];
        t[1] = acc;
      }
    }
  }
  if (threadIdx.x == 0) {
    P.disc[ci] = cl.disc;
    P.maxdisc[ci] = cl.maxdisc;
    P.degen[ci] = cl.degen;
    P.unconv[ci] = cl.unconv;
  }
}

__global__ void init_plus_kernel(double2 *f64, int64_t mps_stride, const int64_t *site_off, const int32_t *pad,
                                 int32_t *dims, int32_t m, int64_t n, const int64_t *base) {
  const int64_t ci = circuit_of(base);
  if (ci >= n) return;
  const double h = 0.70710678118654752440;
  for (int l = threadIdx.x; l <= m; l += blockDim.x) {
    dims[ci * (m + 1) + l] = 1;
    if (l < m) {
      double2 *A = f64 + ci * mps_stride + site_off[l];
      A[0] = make_double2(h, 0.0);                                  // s = 0, a = 0, b = 0
      A[size_t(pad[l]) * pad[l + 1]] = make_double2(h, 0.0);        // s = 1
    }
  }
}

__global__ void normalize_last_kernel(double2 *f64, int64_t mps_stride, const int64_t *site_off,
                                      const int32_t *pad, int32_t m, int64_t n, const int64_t *base) {
  const int64_t ci = circuit_of(base);
  if (ci >= n) return;
  __shared__ double s_red[256];
  double2 *A = f64 + ci * mps_stride + site_off[m - 1];
  const int cnt = 2 * pad[m - 1] * pad[m];
  double acc = 0.0;
  for (int e = threadIdx.x; e < cnt; e += blockDim.x) acc = fma(A[e].x, A[e].x, fma(A[e].y, A[e].y, acc));
  s_red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (int(threadIdx.x) < o) s_red[threadIdx.x] += s_red[threadIdx.x + o];
    __syncthreads();
  }
  const double nrm = s_red[0];
  if (nrm <= 0.0) return;
  const double inv = 1.0 / sqrt(nrm);
  for (int e = threadIdx.x; e < cnt; e += blockDim.x) A[e] = make_double2(A[e].x * inv, A[e].y * inv);
}

// First circuit of the next graph replay (one thread).
__global__ void set_base_kernel(int64_t *base, int64_t v, int64_t add) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *base = add ? *base + v : v;
}

}  // namespace

// FP64 tensors of src copied into dst, whose pads are no larger (and no
// smaller than every bond dimension of src): block (mps i, site l) of dst is
// [s][r][c] with r < dst pad[l], c < dst pad[l+1].  Grid (m, MPS chunk).
__global__ __launch_bounds__(256) void repad_f64_kernel(const double2 *__restrict__ src, double2 *__restrict__ dst,
                                                        const int32_t *__restrict__ spad,
                                                        const int32_t *__restrict__ dpad,
                                                        const int64_t *__restrict__ soff,
                                                        const int64_t *__restrict__ doff, int64_t sstride,
                                                        int64_t dstride, int32_t m, int64_t n) {
  const int l = blockIdx.x;
  const int64_t i = blockIdx.y;
  if (l >= m || i >= n) return;
  const int sl = spad[l], sr = spad[l + 1], dl = dpad[l], dr = dpad[l + 1];
  const double2 *a = src + i * sstride + soff[l];
  double2 *b = dst + i * dstride + doff[l];
  for (int e = threadIdx.x; e < 2 * dl * dr; e += blockDim.x) {
    const int s = e / (dl * dr), r = (e / dr) % dl, c = e % dr;
    b[e] = a[(size_t(s) * sl + r) * sr + c];
  }
}

qk_status launch_repad_f64(const qk_mps_batch *src, qk_mps_batch *dst, hipStream_t stream) {
  if (src->n == 0) return QK_OK;
  for (int l = 0; l <= src->m; ++l)
    if (dst->pad[l] > src->pad[l]) return fail(QK_EINVAL, "repad to a larger pad");
  const int64_t chunk = 65535;
  for (int64_t i0 = 0; i0 < src->n; i0 += chunk) {
    const int64_t cnt = std::min(chunk, src->n - i0);
    hipLaunchKernelGGL(repad_f64_kernel, dim3(unsigned(src->m), unsigned(cnt)), dim3(256), 0, stream,
                       src->f64 + i0 * src->mps_stride, dst->f64 + i0 * dst->mps_stride, src->pad_dev,
                       dst->pad_dev, src->site_off_dev, dst->site_off_dev, src->mps_stride, dst->mps_stride,
                       src->m, cnt);
    QK_HIP_CHECK(hipGetLastError());
  }
  return QK_OK;
}

// The step list shared by every circuit: runs of Rz records, centre moves
// and two-qubit gates in circuit order, then the final moves to the last
// site.  gate_no[i] is the number of two-qubit gates done after step i when
// step i is a gate, and 0 otherwise.
struct SimPlan {
  std::vector<SimStep> steps;
  std::vector<int64_t> gate_no;
  std::vector<int32_t> bond;   // largest bond that any step can leave at each cut
  int size = 2;                // largest Jacobi matrix the bonds allow
  bool wide = false;           // some step may lie next to a bond above kWideFrom
};

SimPlan *make_sim_plan(const std::vector<qk_gate> &gates, int m, int chi, double cutoff) {
  auto *plan = new SimPlan();
  auto &steps = plan->steps;
  auto &gate_no = plan->gate_no;
  int &size = plan->size;
  bool &wide = plan->wide;
  plan->bond.assign(m + 1, 1);
  std::vector<int> next2q(gates.size(), -1);  // site of the next two-qubit gate
  int nxt = -1;
  for (int gi = int(gates.size()) - 1; gi >= 0; --gi) {
    next2q[gi] = nxt;
    if (gates[gi].op != OP_RZ) nxt = gates[gi].site;
  }
  // bond[l]: no circuit's bond can be larger here.  A two-site step leaves
  // at most the rows and columns of its Jacobi matrix, a gate at most chi
  // and, where the cutoff drops rounding noise (weights near 1e-30), the
  // rank of its operator (Rxx: 2, SWAP: 4) times the bond before it.
  std::vector<int> bond(m + 1, 1);
  auto push = [&](SimStep x, int64_t g) {
    if (x.kind == STEP_TWO_SITE) {
      const int Dp = bond[x.p], Dn = bond[x.p + 2];
      int &Dm = bond[x.p + 1];
      const bool right = x.mode == GATE_RIGHT || x.mode == MOVE_RIGHT;
      if (x.mode == MOVE_RIGHT || x.mode == MOVE_LEFT) {
        size = std::max({size, 2 * Dp, 2 * Dn, Dm});
        Dm = std::min(Dm, 2 * (right ? Dp : Dn));
      } else {
        size = std::max({size, 2 * Dp, 2 * Dn});
        const int rank = cutoff > 1e-20 ? (x.op == OP_RXX ? 2 : 4) * Dm : chi;
        Dm = std::min({chi, 2 * Dp, 2 * Dn, rank});
      }
      wide |= Dp > kWideFrom || Dn > kWideFrom;
      x.nr = Dm;
      plan->bond[x.p + 1] = std::max(plan->bond[x.p + 1], Dm);
    }
    steps.push_back(x);
    gate_no.push_back(g);
  };
  int center = 0;
  int64_t d2q = 0;
  size_t gi = 0;
  while (gi < gates.size()) {
    if (gates[gi].op == OP_RZ) {
      size_t ge = gi;
      while (ge < gates.size() && gates[ge].op == OP_RZ) ++ge;
      push({STEP_RZ, 0, 0, 0, -1, -1, int32_t(gi), int32_t(ge - gi), 0, 0, 0, 0, 0, 0}, 0);
      gi = ge;
      continue;
    }
    const int p = gates[gi].site;
    for (; center < p; ++center) push({STEP_TWO_SITE, center, MOVE_RIGHT, OP_ID, -1, -1, -1, 0, 0, 0, 0, 0, 0, 0}, 0);
    for (; center > p + 1; --center) push({STEP_TWO_SITE, center - 1, MOVE_LEFT, OP_ID, -1, -1, -1, 0, 0, 0, 0, 0, 0, 0}, 0);
    const bool absorb_right = next2q[gi] < 0 || next2q[gi] > p;
    push({STEP_TWO_SITE, p, absorb_right ? GATE_RIGHT : GATE_LEFT, gates[gi].op == 1 ? OP_RXX : OP_SWAP,
          gates[gi].feat_i, gates[gi].feat_j, int32_t(d2q), 0, 0, 0, 0, 0, 0, 0},
         d2q + 1);
    ++d2q;
    center = absorb_right ? p + 1 : p;
    ++gi;
  }
  for (; center < m - 1; ++center) push({STEP_TWO_SITE, center, MOVE_RIGHT, OP_ID, -1, -1, -1, 0, 0, 0, 0, 0, 0, 0}, 0);
  return plan;
}
void free_sim_plan(SimPlan *plan) { delete plan; }
const std::vector<int32_t> &sim_plan_bonds(const SimPlan *plan) { return plan->bond; }

qk_status run_simulation(qk_mps_batch *b, const SimPlan *plan, const double *features_dev,
                         const std::vector<qk_gate> &gates, const qk_circuit_spec &spec, int chi, double cutoff, hipStream_t stream, qk_progress_fn fn,
                         void *user, int64_t every, int64_t graph_circuits, int32_t *trace) {
  const int64_t n = b->n;
  const int m = b->m;
  int n2q = 0;
  for (const auto &g : gates) n2q += g.op != OP_RZ ? 1 : 0;
  b->n_two_qubit_gates = n2q;
  if (n == 0) return QK_OK;
  if (n > 0x7fffffff) return fail(QK_EINVAL, "too many points for one launch");
  if (graph_circuits > 0 && fn) return fail(QK_EINVAL, "progress callbacks are not available with graph replay");

  // reject non-finite features before any launch
  {
    std::vector<double> xh(size_t(n) * m);
    QK_HIP_CHECK(hipMemcpyAsync(xh.data(), features_dev, sizeof(double) * xh.size(), hipMemcpyDeviceToHost, stream));
    QK_HIP_CHECK(hipStreamSynchronize(stream));
    for (double v : xh)
      if (!std::isfinite(v)) return fail(QK_EINVAL, "non-finite feature value");
  }

  // Graph mode: one graph records the launches that simulate `grid` circuits
  // from start to end and is replayed until every circuit is done; otherwise
  // the launches cover the whole batch.
  const bool graph = graph_circuits > 0;
  const int64_t grid = graph ? std::min(n, graph_circuits) : n;
  const int64_t replays = (n + grid - 1) / grid;

  std::vector<SimStep> steps = plan->steps;
  for (SimStep &x : steps)
    if (x.kind == STEP_TWO_SITE) {
      x.Pp = b->pad[x.p];
      x.Pm = b->pad[x.p + 1];
      x.Pn = b->pad[x.p + 2];
      x.off_p = b->site_off[x.p];
      x.off_q = b->site_off[x.p + 1];
    }
  const auto &gate_no = plan->gate_no;
  const int size = plan->size;
  const bool wide = plan->wide;

  // Device buffers: gate records, step list, SVD scratch of one slot per
  // workgroup of a launch, and (graph mode) the first circuit of a replay.
  const DevAlloc al = allocator_for_current_device();
  const int nk = size <= 16 ? 16 : size <= 32 ? 32 : size <= 64 ? 64 : kSvMaxN;
  const size_t steps_bytes = sizeof(SimStep) * steps.size(), recs_bytes = sizeof(qk_gate) * gates.size();
  // [parameters | steps | gate records | first circuit of a replay]
  const size_t steps_at = (sizeof(SvParams) + 15) / 16 * 16, recs_at = steps_at + steps_bytes;
  const size_t base_at = (recs_at + recs_bytes + 15) / 16 * 16, block_bytes = base_at + 16;
  void *block = nullptr, *scratch = nullptr, *wscratch = nullptr;
  auto release = [&]() {
    for (void *ptr : {block, scratch, wscratch})
      if (ptr) dev_free(al, ptr, stream, true);
  };
  block = dev_alloc(al, block_bytes, stream, true);
  if (nk > 32) scratch = dev_alloc(al, sizeof(double2) * nk * nk * size_t(grid), stream, true);
  if (wide) wscratch = dev_alloc(al, sizeof(double2) * kWideSlot * size_t(grid), stream, true);
  if (!block || (nk > 32 && !scratch) || (wide && !wscratch)) {
    release();
    return fail(QK_ENOMEM, "device allocation of the simulation buffers failed");
  }
  auto *block8 = static_cast<uint8_t *>(block);
  const auto *params = reinterpret_cast<const SvParams *>(block8);
  const auto *steps_d = reinterpret_cast<const SimStep *>(block8 + steps_at);
  const auto *recs = reinterpret_cast<const qk_gate *>(block8 + recs_at);
  auto *base = graph ? reinterpret_cast<int64_t *>(block8 + base_at) : nullptr;

  SvParams P{};
  P.f64 = b->f64;
  P.mps_stride = b->mps_stride;
  P.site_off = b->site_off_dev;
  P.pad = b->pad_dev;
  P.dims = b->dims_dev;
  P.m = m;
  P.chi = chi;
  P.gate_split = spec.gate_split;
  P.coef_xx = spec.coef_xx;
  P.cutoff = cutoff;
  P.X = features_dev;
  P.ldx = m;
  P.scratch = static_cast<double2 *>(scratch);
  P.scratch_stride = int64_t(nk) * nk;
  P.wscratch = static_cast<double2 *>(wscratch);
  P.disc = b->disc_dev;
  P.maxdisc = b->maxdisc_dev;
  P.degen = b->degen_dev;
  P.unconv = b->unconv_dev;
  P.n = n;
  P.trace = trace;
  P.trace_n2q = n2q;
  P.base = base;
  {
    std::vector<uint8_t> host(block_bytes, 0);
    std::memcpy(host.data(), &P, sizeof(P));
    if (steps_bytes) std::memcpy(host.data() + steps_at, steps.data(), steps_bytes);
    if (recs_bytes) std::memcpy(host.data() + recs_at, gates.data(), recs_bytes);
    const qk_status up = upload(block, host.data(), block_bytes, stream);
    if (up != QK_OK) {
      release();
      return up;
    }
  }

  // The launches of one pass over `grid` circuits on stream s: the |+>
  // state, the step list in launches of at most kMaxChunkSteps steps (a
  // launch also ends where a progress callback is due), the normalisation of
  // the last site, and in graph mode the advance of the first circuit.
  constexpr size_t kMaxChunkSteps = 256;
  auto pass = [&](hipStream_t s) -> qk_status {
    hipLaunchKernelGGL(init_plus_kernel, dim3(unsigned(grid)), dim3(64), 0, s, b->f64, b->mps_stride,
                       b->site_off_dev, b->pad_dev, b->dims_dev, m, n, P.base);
    if (hipGetLastError() != hipSuccess) return fail(QK_EDEVICE, "initial-state launch failed");
    size_t s0 = 0;
    while (s0 < steps.size()) {
      size_t s1 = s0;
      bool report = false;
      while (s1 < steps.size() && s1 - s0 < kMaxChunkSteps) {
        const int64_t g = gate_no[s1++];
        if (g > 0 && fn && every > 0 && g % every == 0) {
          report = true;
          break;
        }
      }
      auto launch = [&](auto kern, int threads, size_t lds) {
        hipLaunchKernelGGL(kern, dim3(unsigned(grid)), dim3(threads), lds, s, params, steps_d, int(s0), int(s1), recs,
                           spec.coef_z);
      };
      if (nk == 16) launch(sim_steps_kernel<16>, 64 * sim_waves(16), sim_lds_bytes<16>());
      else if (nk == 32) launch(sim_steps_kernel<32>, 64 * sim_waves(32), sim_lds_bytes<32>());
      else if (nk == 64) launch(sim_steps_kernel<64>, 64 * sim_waves(64), sim_lds_bytes<64>());
      else launch(sim_steps_kernel<128>, 64 * sim_waves(128), sim_lds_bytes<128>());
      if (hipGetLastError() != hipSuccess) return fail(QK_EDEVICE, "simulation launch failed");
      if (report) {
        if (hipStreamSynchronize(s) != hipSuccess) return fail(QK_EDEVICE, "simulation step failed");
        if (fn(gate_no[s1 - 1], n2q, user) != 0)
          return fail(QK_EABORTED, "simulation aborted by the progress callback");
      }
      s0 = s1;
    }
    hipLaunchKernelGGL(normalize_last_kernel, dim3(unsigned(grid)), dim3(256), 0, s, b->f64, b->mps_stride,
                       b->site_off_dev, b->pad_dev, m, n, P.base);
    if (hipGetLastError() != hipSuccess) return fail(QK_EDEVICE, "normalisation launch failed");
    if (graph) {
      hipLaunchKernelGGL(set_base_kernel, dim3(1), dim3(64), 0, s, base, grid, int64_t(1));
      if (hipGetLastError() != hipSuccess) return fail(QK_EDEVICE, "replay-advance launch failed");
    }
    return QK_OK;
  };

  qk_status st = QK_OK;
  if (!graph) {
    st = pass(stream);
  } else {
    // The pass is recorded by stream capture on a private stream (the
    // caller's stream may be the legacy null stream, which cannot be
    // captured) and replayed `replays` times there; events order the
    // private stream after the caller's earlier work and the caller's stream
    // after the replays.  The first circuit starts at 0 (a kernel, not a
    // memset, so that the sequence could itself be captured).
    hipLaunchKernelGGL(set_base_kernel, dim3(1), dim3(64), 0, stream, base, int64_t(0), int64_t(0));
    if (hipGetLastError() != hipSuccess) {
      release();
      return fail(QK_EDEVICE, "replay-start launch failed");
    }
    hipStream_t cap = nullptr;
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    hipGraph_t g = nullptr;
    hipGraphExec_t exec = nullptr;
    if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&ev_out, hipEventDisableTiming) != hipSuccess ||
        hipEventRecord(ev_in, stream) != hipSuccess || hipStreamWaitEvent(cap, ev_in, 0) != hipSuccess) {
      st = fail(QK_EDEVICE, "graph stream set-up failed");
    } else if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
      st = fail(QK_EDEVICE, "graph capture failed to start");
    } else {
      st = pass(cap);
      // the capture is ended on every path so that the stream stays usable
      const hipError_t ce = hipStreamEndCapture(cap, &g);
      if (st == QK_OK && ce != hipSuccess) st = fail(QK_EDEVICE, std::string("graph capture failed: ") + hipGetErrorString(ce));
      if (st == QK_OK) {
        const hipError_t ie = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
        if (ie != hipSuccess) st = fail(QK_EDEVICE, std::string("graph instantiation failed: ") + hipGetErrorString(ie));
      }
      for (int64_t r = 0; st == QK_OK && r < replays; ++r) {
        const hipError_t le = hipGraphLaunch(exec, cap);
        if (le != hipSuccess) st = fail(QK_EDEVICE, std::string("graph launch failed: ") + hipGetErrorString(le));
      }
    }
    if (cap) {
      // the caller's stream continues after the replays
      if (ev_out && hipEventRecord(ev_out, cap) == hipSuccess) (void)hipStreamWaitEvent(stream, ev_out, 0);
      (void)hipStreamSynchronize(cap);
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    if (g) (void)hipGraphDestroy(g);
    if (ev_in) (void)hipEventDestroy(ev_in);
    if (ev_out) (void)hipEventDestroy(ev_out);
    if (cap) (void)hipStreamDestroy(cap);
  }
  release();
  if (st != QK_OK) {
    (void)hipStreamSynchronize(stream);
    return st;
  }
  QK_HIP_CHECK(hipStreamSynchronize(stream));
  if (fn && fn(n2q, n2q, user) != 0) return fail(QK_EABORTED, "simulation aborted by the progress callback");
  return QK_OK;
}

}  // namespace qk
