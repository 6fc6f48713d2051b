// Sparse direct solve of the masked K (multifrontal, FP64): numeric phase.
//
// Sec. 2.2.2 of the paper solves K u = f with direct solvers.  The plan (direct_plan.cpp) holds
// the fronts of a nested dissection: front F has own DOFs S (eliminated there) and boundary DOFs
// B.  Its matrix is the blocks of K with a column in S, plus the children's Schur complements;
// eliminating S gives
//   W = F_SS^-1,  G = F_BS W,  U = F_BB - G F_SB     (U goes to the parent),
// and a right-hand side passes up and down the tree with two products a front:
//   up:    b_S = f_S + children's v,  v_B = children's v - G b_S
//   down:  x_S = W b_S - G^T x_B.
// W is kept as a full matrix instead of a triangular factor: a substitution is then one product
// over the front's stored panel, one launch a level, instead of a chain of triangular steps.
//
// F_SS is inverted by the symmetric sweep operator on panels of DIRECT_NB columns.  A sweep of
// panel J with D = F_JJ takes every row I of the front's columns through
//   F_IK -= (F_IJ D^-1) F_KJ^T,  F_IJ = F_IJ D^-1,  F_JK = its transpose,  F_JJ = -D^-1,
// after which the own rows hold -W and the boundary rows G.  A level's panels are a chain of
// launches: launch q scales panel q (F_IJ D^-1 into a buffer of its own) and updates all columns
// with panel q - 1; what the scaling needs of that update it forms itself, one more product of
// tiles, so that a panel costs one launch instead of two.  The first launch assembles the columns,
// the last update goes with the Schur complements.  Sweeps alternate between two copies of the
// columns and of the scaled panel, so no work item reads what another one of the same launch
// writes.  The products run on the matrix cores (v_mfma_f64_16x16x4_f64) from LDS tiles.  All fronts of one level share the launches; the items
// of a launch come from the plan, so a front's arithmetic does not depend on what else is in the
// launch.  No atomics: every entry has one writer and a fixed order of additions.
#include <cmath>

#include "sso_internal.h"
#include "wave.h"

namespace sso {
namespace {

constexpr int NB = DIRECT_NB;
constexpr int TPB = 256;
constexpr int KC = 32;                // depth of an LDS tile
constexpr int LDK = KC + 1;           // its row length: odd, so that 16 rows spread over the banks
constexpr int LDN = NB + 1;
constexpr int FWD_LANES = TPB / DIRECT_FWD_ROWS;    // lanes of a row
constexpr int BWD_TPB = 512;
constexpr int BWD_GROUPS = BWD_TPB / DIRECT_BWD_COLS;
constexpr int BWD_CHUNK = 2048;       // rows of the vector staged at a time
// A pivot below this share of K's diagonal entry means that K is singular to working precision
// (rounding leaves some 1e-15 of it in place of a zero pivot); the solve then goes back to PCG.
constexpr double PIVOT_MIN = 1e-13;

// The wave's number in its workgroup, in a scalar register.
__device__ __forceinline__ int wave_id() {
  return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
}

// The lane's number, computed anew here: what follows from it is then not carried in registers
// through a caller's loop.
__device__ __forceinline__ int lane_here() {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}

typedef double d4 __attribute__((ext_vector_type(4)));

// The item of this workgroup, or false past the end of the problem's list.  probs == nullptr: one
// problem, given by value with its list's offset; else problem blockIdx.y, whose list is looked up.
__device__ __forceinline__ bool take_item(DirectArgs& a, const DirectArgs* __restrict__ probs,
                                          int first, int level, int step, DirectItem& it) {
  if (probs) {
    a = probs[blockIdx.y];
    if (level >= a.n_levels) return false;
    if (step >= STEP_PANEL && step - STEP_PANEL > a.level_np[level]) return false;
    const DirectRange r = a.steps[a.level_off[level] + step];
    if ((int)blockIdx.x >= r.cnt) return false;
    first = r.off;
  }
  it = a.items[first + (int)blockIdx.x];
  return true;
}

// A child's Schur complement (its lower triangle is stored).  at(r, c): the entry at DOF rows r, c
// of its boundary, 0 where either is negative (not in the boundary).  Loads are unconditional, from
// entry 0 then, so that a thread's loads are all in flight together; the byte offset fits 32 bits
// (DIRECT_MAX_BOUNDARY), which leaves the base in scalar registers.
struct ChildU {
  const double* __restrict__ u;
  __device__ __forceinline__ double at(int r, int c) const {
    const bool in = (r | c) >= 0;
    const unsigned hi = r > c ? r : c, lo = r > c ? c : r;
    const unsigned e = in ? hi * (hi + 1) / 2 + lo : 0u;
    const double v =
        *reinterpret_cast<const double*>(reinterpret_cast<const char*>(u) + (e * 8u));
    return in ? v : 0.0;
  }
};

// Where a front's sweep p reads and writes its columns: the last one writes the factor, the ones
// before alternate, the first reads the assembled front.
__device__ __forceinline__ double* sweep_dst(const DirectArgs& a, const DirectFront& F, int p) {
  return ((F.np - 1 - p) & 1) == 0 ? a.fact + F.fact_off : a.x1 + F.again_off;
}
__device__ __forceinline__ const double* sweep_src(const DirectArgs& a, const DirectFront& F,
                                                   int p) {
  return p == 0 ? a.f0 + F.work_off : sweep_dst(a, F, p - 1);
}

// Up to 64 rows x KC columns of a row-major array on their way into an LDS tile, zero outside.
// 16-byte loads: rows start at even offsets (every row length is a multiple of 6 or 64), and the
// number of columns is even, so a pair lies inside or outside as a whole.
struct TileLoad {
  static constexpr int PER = NB * KC / 2 / TPB;
  double2 v[PER];
  __device__ __forceinline__ void load(const double* __restrict__ src, int64_t ld, int rows,
                                       int k0, int kn) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = (int)threadIdx.x + u * TPB, r = e / (KC / 2), c = 2 * (e % (KC / 2));
      v[u] = double2{0.0, 0.0};
      if (r < rows && k0 + c < kn)
        v[u] = *reinterpret_cast<const double2*>(src + (int64_t)r * ld + k0 + c);
    }
  }
  __device__ __forceinline__ void store(double* dst) const {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = (int)threadIdx.x + u * TPB, r = e / (KC / 2), c = 2 * (e % (KC / 2));
      dst[r * LDK + c] = v[u].x;
      dst[r * LDK + c + 1] = v[u].y;
    }
  }
};

// acc += A B^T over kn columns of LDS tiles A, B (64 rows each): the wave's 32 x 32 quadrant as
// 2 x 2 matrix-core tiles.
__device__ __forceinline__ void mma_tile(const double* A, int lda, const double* B, int ldb,
                                         int kn, d4 acc[2][2]) {
  const int lane = lane_here(), wave = wave_id();
  const int l16 = lane & 15, kq = lane >> 4;
  const double* pa = A + (32 * (wave >> 1) + l16) * lda + kq;
  const double* pb = B + (32 * (wave & 1) + l16) * ldb + kq;
  auto step = [&](int k) {
    const double a0 = pa[k], a1 = pa[16 * lda + k];
    const double b0 = pb[k], b1 = pb[16 * ldb + k];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  };
  if (kn == KC) {
#pragma unroll
    for (int k = 0; k < KC; k += 4) step(k);
  } else {
    for (int k = 0; k < kn; k += 4) step(k);
  }
}

// acc += A B^T, both row-major in memory, over kn columns: the next KC columns are on their way
// while the matrix cores work on the ones in LDS (as, bs: NB x LDK each).  From column split on, a
// multiple of KC, A and B are rows of NB in A2 and B2.
__device__ __forceinline__ void product(const double* __restrict__ A, int64_t lda, int ra,
                                        const double* __restrict__ B, int64_t ldb, int rb, int kn,
                                        double* as, double* bs, d4 acc[2][2], int split,
                                        const double* __restrict__ A2,
                                        const double* __restrict__ B2) {
  TileLoad ta, tb;
  for (int k0 = 0; k0 < kn; k0 += KC) {
    auto fetch = [&](int k) {
      const bool second = k >= split;
      const int64_t la = second ? NB : lda, lb = second ? NB : ldb;
      ta.load(second ? A2 - split : A, la, ra, k, kn);
      tb.load(second ? B2 - split : B, lb, rb, k, kn);
    };
    if (k0)
      __syncthreads();
    else
      fetch(0);
    ta.store(as);
    tb.store(bs);
    __syncthreads();
    if (k0 + KC < kn) fetch(k0 + KC);
    mma_tile(as, LDK, bs, LDK, kn - k0 < KC ? kn - k0 : KC, acc);
  }
}

__device__ __forceinline__ void product(const double* __restrict__ A, int64_t lda, int ra,
                                        const double* __restrict__ B, int64_t ldb, int rb, int kn,
                                        double* as, double* bs, d4 acc[2][2]) {
  TileLoad ta, tb;
  ta.load(A, lda, ra, 0, kn);
  tb.load(B, ldb, rb, 0, kn);
  for (int k0 = 0; k0 < kn; k0 += KC) {
    if (k0) __syncthreads();
    ta.store(as);
    tb.store(bs);
    __syncthreads();
    if (k0 + KC < kn) {
      ta.load(A, lda, ra, k0 + KC, kn);
      tb.load(B, ldb, rb, k0 + KC, kn);
    }
    mma_tile(as, LDK, bs, LDK, kn - k0 < KC ? kn - k0 : KC, acc);
  }
}

// f(row, column, value) over the wave's accumulators: lane l holds column l % 16 and rows
// l / 16 + 4 v of each 16 x 16 tile.
template <class Fn>
__device__ __forceinline__ void each_acc(const d4 acc[2][2], Fn f) {
  const int lane = lane_here(), wave = wave_id();
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        f(32 * (wave >> 1) + 16 * i + (lane >> 4) + 4 * v, 32 * (wave & 1) + 16 * j + (lane & 15),
          acc[i][j][v]);
}

__device__ __forceinline__ void clear(d4 acc[2][2]) {
  for (int i = 0; i < 2; ++i)
    for (int j = 0; j < 2; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
}

// 1 / x for a pivot: the hardware's estimate and two Newton steps (relative error some 1e-16).
__device__ __forceinline__ double reciprocal(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
  return r;
}

// d[j] += t * (lane K's d[j], of each row of 16 lanes) for all j but K, d[K + 1] first: the next
// step waits for it.  One instruction an entry, the broadcast being a DPP control of the multiply-
// add; the compiler makes a move and a multiply-add of it, through one pair of registers (253
// cycles a step instead of 154).  The waits are those that DPP asks for after a write of its source.
template <int K>
__device__ __forceinline__ void sweep_update(double (&d)[16], double t) {
#define SSO_FMA(n) "v_fmac_f64_dpp %" #n ", %" #n ", %15 row_newbcast:%c16 row_mask:0xf bank_mask:0xf\n"
#define SSO_ARG(n) "+&v"(d[(K + 1 + n) & 15])
  asm("s_nop 1\n" SSO_FMA(0) SSO_FMA(1) SSO_FMA(2) SSO_FMA(3) SSO_FMA(4) SSO_FMA(5) SSO_FMA(6)
          SSO_FMA(7) SSO_FMA(8) SSO_FMA(9) SSO_FMA(10) SSO_FMA(11) SSO_FMA(12) SSO_FMA(13)
              SSO_FMA(14) "s_nop 1"
      : SSO_ARG(0), SSO_ARG(1), SSO_ARG(2), SSO_ARG(3), SSO_ARG(4), SSO_ARG(5), SSO_ARG(6),
        SSO_ARG(7), SSO_ARG(8), SSO_ARG(9), SSO_ARG(10), SSO_ARG(11), SSO_ARG(12), SSO_ARG(13),
        SSO_ARG(14)
      : "v"(t), "n"(K));
#undef SSO_FMA
#undef SSO_ARG
}

// Steps K .. 15 of the sweep of a symmetric 16 x 16 block, row l of it in lane l of each row of 16
// lanes.  A row is left times its pivot from its step on (in a sweep only the rows still to come
// are read by others), so that a step is one multiply-add an entry and no selection.
template <int K>
__device__ __forceinline__ void sweep_steps(double (&d)[16], int l16, double& pivot) {
  if constexpr (K < 16) {
    const double p = dpp_move<0x150 + K>(d[K]);          // row_newbcast
    const double x = __builtin_amdgcn_rcp(p);
    const bool me = l16 == K;
    const double c = me ? 0.0 : -d[K];
    if (me) pivot = p;
    const double e = __builtin_fma(-p, x, 1.0);          // 1 / p = x (1 + e + e^2)
    const double c0 = c * x;
    const double t = __builtin_fma(c0, __builtin_fma(e, e, e), c0);
    sweep_update<K>(d, t);
    d[K] = me ? -1.0 : -t;
    sweep_steps<K + 1>(d, l16, pivot);
  }
}

constexpr int LDS16 = 18;     // row length of 16 columns in LDS: 16-byte reads, spread over the banks
constexpr int SWEEP_PANEL = (NB + 16) * LDS16;
constexpr int SWEEP_LDS = 2 * SWEEP_PANEL;      // two panels alternate

// Sweeps the leading nb columns of a 64 x 64 symmetric block, held as matrix-core accumulators
// (each_acc's layout): the block becomes minus its inverse; pivot[k], k < nb rounded up to 16, are
// the pivots.  The workgroup enters with lds free and pivot unused, and leaves with lds free.
//
// Panels of 16 columns: the wave that holds the pivot block inverts it by itself, register to
// register; the others publish the panel's columns meanwhile; and all update their tiles on the
// matrix cores.  The product -F D^-1 comes out transposed, which is the order of the next product's
// left operand, and an accumulator of a symmetric block that of its right one, so nothing goes
// through LDS in between.  The next pivot block is updated first and inverted while the other waves
// go on.  A block takes 8.3 us at 2.4 GHz, most of it in the chain of the four inversions, 16 steps
// of 154 cycles each (issue-bound); 9.3 us with the update in front of the next inversion; 20 us
// swept one column at a time, each published through LDS with a barrier.
__device__ __forceinline__ void sweep(d4 d[2][2], int nb, double* lds, double* pivot) {
  const int lane = lane_here();
  const int wave = wave_id();
  const int l16 = lane & 15, kq = lane >> 4, wr = wave >> 1, wc = wave & 1;
  auto four = [](const double* q, double (&o)[4]) {
    const double2 y = *reinterpret_cast<const double2*>(q);
    const double2 z = *reinterpret_cast<const double2*>(q + 2);
    o[0] = y.x;
    o[1] = y.y;
    o[2] = z.x;
    o[3] = z.y;
  };
  // the panel's columns, column c at 4 (c % 4) + c / 4; then minus the pivot block's inverse
  auto panel = [&](int s) { return lds + s * SWEEP_PANEL; };
  auto invert = [&](const d4& block, int first, int s) {
    double* T = panel(s) + first * LDS16;        // nothing else of the panel lies here
    double* D = panel(s) + NB * LDS16;
#pragma unroll
    for (int v = 0; v < 4; ++v) T[l16 * LDS16 + kq + 4 * v] = block[v];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double x[16];
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
      const double2 y = *reinterpret_cast<const double2*>(T + l16 * LDS16 + j);
      x[j] = y.x;
      x[j + 1] = y.y;
    }
    double p = 1.0;
    sweep_steps<0>(x, l16, p);
    const double inv = reciprocal(p);
    if (kq == 0) {
      pivot[first + l16] = p;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int v = 0; v < 4; v += 2)
          *reinterpret_cast<double2*>(D + l16 * LDS16 + 4 * g + v) =
              double2{x[g + 4 * v] * inv, x[g + 4 * v + 4] * inv};
    }
  };
  auto publish = [&](int half, const int s) {
    if (wc != half) return;
    const int at = 4 * (l16 & 3) + (l16 >> 2);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (wr == half && i == s) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        panel(s)[(32 * wr + 16 * i + kq + 4 * v) * LDS16 + at] = d[i][s][v];
    }
  };
  if (wave == 0) invert(d[0][0], 0, 0);
  publish(0, 0);
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (32 * half + 16 * s >= nb) break;
      const int next_half = half + s, n = s ^ 1, next = 32 * next_half + 16 * n;
      __syncthreads();
      const double* P = panel(s);
      double inv[4], row[2][4], col[2][4];
      four(P + (NB + l16) * LDS16 + 4 * kq, inv);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        four(P + (32 * wr + 16 * i + l16) * LDS16 + 4 * kq, row[i]);
        four(P + (32 * wc + 16 * i + l16) * LDS16 + 4 * kq, col[i]);
      }
      d4 w[2];                                   // minus the scaled rows, transposed
      auto scale = [&](const int i) {
        if (wr == half && i == s) return;
        w[i] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v)
          w[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(inv[v], row[i][v], w[i], 0, 0, 0);
      };
      auto update = [&](const int i, const int j) {
        const bool in_row = wr == half && i == s, in_col = wc == half && j == s;
        if (in_row && in_col) {
          d[i][j] = d4{inv[0], inv[1], inv[2], inv[3]};
        } else if (in_row && wr == wc) {
          d[i][j] = -w[j];
        } else if (in_row || in_col) {
          d4 x = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int v = 0; v < 4; ++v)
            x = __builtin_amdgcn_mfma_f64_16x16x4f64(in_row ? inv[v] : row[i][v],
                                                     in_row ? col[j][v] : inv[v], x, 0, 0, 0);
          d[i][j] = -x;
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            d[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i][v], col[j][v], d[i][j], 0, 0, 0);
        }
      };
      scale(n);
      update(n, n);
      if (next < nb && wr == next_half && wc == next_half) invert(d[n][n], next, n);
      scale(s);
      update(n, s);
      update(s, n);
      update(s, s);
      if (next < nb) publish(next_half, n);
    }
  }
  __syncthreads();
}

constexpr int POOL = 3 * NB * LDK;    // doubles of LDS that the panel kernels cut their tiles from
static_assert(NB * LDN + NB * LDK <= POOL, "the inverse and a tile of the row tile fit");
static_assert(SWEEP_LDS <= POOL, "the sweep's panel fits");

// The scaled panel of step q: q even and odd alternate.  After both, the last panel's columns
// before they are scaled, boundary tiles only.
__device__ __forceinline__ double* scaled(const DirectArgs& a, const DirectFront& F, int q, int i) {
  return a.w + F.w_off + ((int64_t)(q & 1) * F.nt + i) * NB * NB;
}
__device__ __forceinline__ double* unscaled(const DirectArgs& a, const DirectFront& F, int i) {
  return a.w + F.w_off + (2 * (int64_t)F.nt + i - F.np) * NB * NB;
}

// Sets the flag where a pivot of the nb from own DOF j0 on is too small.
__device__ __forceinline__ void check_pivots(const DirectArgs& a, const DirectFront& F, int j0,
                                             int nb, const double* pivots) {
  if ((int)threadIdx.x >= nb) return;
  const int r = j0 + (int)threadIdx.x, n = r / 6;
  const double k = a.K[36 * (int64_t)a.bdiag[a.nodes[F.nodes_off + n]] + 7 * (r - 6 * n)];
  if (!(pivots[threadIdx.x] > PIVOT_MIN * k)) atomicOr(a.flag, 1u);
}

// Panel q > 0 of a front scaled, row tile i: D^-1 of its pivot block (by every workgroup of the
// front for itself, which takes no longer than one of them doing it for the others) and F_IJ D^-1,
// both first brought up to date with panel q - 1.
__device__ __forceinline__ void scale_tile(const DirectArgs& a, const DirectFront& F, int q, int i,
                                           double* pool, double* pivots) {
  const int64_t ld = F.ns6;
  const int j0 = q * NB;
  const int nb = F.ns6 - j0 < NB ? F.ns6 - j0 : NB;
  const DirectRows R = direct_rows(F, i);
  const bool pivot = i == q;
  const double* __restrict__ src = sweep_src(a, F, q - 1);
  // the pivot block and the row tile as accumulators (identity past the last column)
  d4 d[2][2], f[2][2];
  const int lane = threadIdx.x & 63, wave = wave_id();
  const bool swept = i == q - 1;   // rows of the panel before: its scaled tile, transposed
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 32 * (wave >> 1) + 16 * u + (lane >> 4) + 4 * v;
        const int c = 32 * (wave & 1) + 16 * w + (lane & 15);
        d[u][w][v] = r < nb && c < nb ? src[(int64_t)(j0 + r) * ld + j0 + c] : (r == c ? 1.0 : 0.0);
        f[u][w][v] = 0.0;
        if (!pivot && r < R.n && c < nb)
          f[u][w][v] = swept ? scaled(a, F, q - 1, q)[c * NB + r]
                             : src[(int64_t)(R.r0 + r) * ld + j0 + c];
      }
  double* ws = pool;                    // scaled rows of the pivot block
  double* wi = pool + NB * LDK;         // scaled rows of the row tile
  double* cs = pool + 2 * NB * LDK;     // the pivot rows' entries in the panel before
  TileLoad tw, ti, tc;
  const double* __restrict__ pw = scaled(a, F, q - 1, q);
  const double* __restrict__ pi = scaled(a, F, q - 1, i);
  const double* __restrict__ pc = src + (int64_t)j0 * ld + j0 - NB;
  const bool row = !pivot && !swept;
  d4 ud[2][2], uf[2][2];
  clear(ud);
  clear(uf);
  tw.load(pw, NB, nb, 0, NB);
  tc.load(pc, ld, nb, 0, NB);
  if (row) ti.load(pi, NB, R.n, 0, NB);
  for (int k0 = 0; k0 < NB; k0 += KC) {
    if (k0) __syncthreads();
    tw.store(ws);
    tc.store(cs);
    if (row) ti.store(wi);
    __syncthreads();
    if (k0 + KC < NB) {
      tw.load(pw, NB, nb, k0 + KC, NB);
      tc.load(pc, ld, nb, k0 + KC, NB);
      if (row) ti.load(pi, NB, R.n, k0 + KC, NB);
    }
    mma_tile(ws, LDK, cs, LDK, KC, ud);
    if (row) mma_tile(wi, LDK, cs, LDK, KC, uf);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      d[u][w] -= ud[u][w];
      if (row) f[u][w] -= uf[u][w];
    }
  if (q == F.np - 1 && i >= F.np) {     // for the Schur step
    double* X = unscaled(a, F, i);
    each_acc(f, [&](int r, int c, double v) {
      if (r < R.n && c < nb) X[r * NB + c] = v;
    });
  }
  __syncthreads();     // the pool is free
  sweep(d, nb, pool, pivots);
  double* out = scaled(a, F, q, i);
  if (pivot) {
    check_pivots(a, F, j0, nb, pivots);
    each_acc(d, [&](int r, int c, double v) {
      if (r < nb && c < nb) out[r * NB + c] = -v;
    });
    return;
  }
  double* ds = pool;
  double* fs = pool + NB * LDN;
  each_acc(d, [&](int r, int c, double v) { ds[r * LDN + c] = -v; });
  d4 acc[2][2];
  clear(acc);
#pragma unroll
  for (int h = 0; h < 2; ++h) {      // columns 32 h .. of the row tile: the waves of that half
    if (32 * h >= nb) break;
    if (h) __syncthreads();
    if ((wave & 1) == h)
      each_acc(f, [&](int r, int c, double v) { fs[r * LDK + c - 32 * h] = v; });
    __syncthreads();
    const int kn = nb - 32 * h < KC ? nb - 32 * h : KC;
    mma_tile(fs, LDK, ds + 32 * h, LDN, kn, acc);
  }
  each_acc(acc, [&](int r, int c, double v) {
    if (r < R.n && c < nb) out[r * NB + c] = v;
  });
}

// Tile (i, j) of a front's columns from one copy to the other, with panel p.
__device__ __forceinline__ void update_tile(const DirectArgs& a, const DirectFront& F, int p, int i,
                                            int j, double* pool) {
  const double* __restrict__ src = sweep_src(a, F, p);
  double* __restrict__ dst = sweep_dst(a, F, p);
  const int64_t ld = F.ns6;
  const int j0 = p * NB;
  const int nb = F.ns6 - j0 < NB ? F.ns6 - j0 : NB;
  const DirectRows R = direct_rows(F, i);
  const int c0 = j * NB;
  const int nc = F.ns6 - c0 < NB ? F.ns6 - c0 : NB;
  const double* __restrict__ wi = scaled(a, F, p, i);
  if (j == p || i == p) {
    // the panel's own column (F_IJ D^-1, -D^-1 on the diagonal) and row (its transpose)
    const double* __restrict__ wj = scaled(a, F, p, j);
    for (int e = threadIdx.x; e < NB * NB; e += TPB) {
      const int r = e / NB, c = e - r * NB;
      if (r >= R.n || c >= nc) continue;
      const double v = j == p ? (i == p ? -wi[r * NB + c] : wi[r * NB + c]) : wj[c * NB + r];
      dst[(int64_t)(R.r0 + r) * ld + c0 + c] = v;
    }
    return;
  }
  d4 f[2][2], acc[2][2];
  const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = 32 * (wave >> 1) + 16 * u + (lane >> 4) + 4 * v;
        const int c = 32 * (wave & 1) + 16 * w + (lane & 15);
        f[u][w][v] = r < R.n && c < nc ? src[(int64_t)(R.r0 + r) * ld + c0 + c] : 0.0;
      }
  clear(acc);
  product(wi, NB, R.n, src + (int64_t)c0 * ld + j0, ld, nc, nb, pool, pool + NB * LDK, acc);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 2; ++w) f[u][w] -= acc[u][w];
  each_acc(f, [&](int r, int c, double v) {
    if (r < R.n && c < nc) dst[(int64_t)(R.r0 + r) * ld + c0 + c] = v;
  });
}

// Step q > 0 of a level's panels: panel q scaled, all columns updated with panel q - 1.
//
// Bound by the scaling's chain, 22 us: 2 for its loads, 4 in the two products that bring the pivot
// block and the row tile up to date (one CU, 74 cycles a matrix instruction), 8.3 in the pivot block's
// inversion, 2.7 in the scaling product, the launch.  With the inversion a column at a time it took
// 33; as two launches, one for the scaling, 10 more.
__global__ void __launch_bounds__(TPB, 2)
k_front_panel(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level, int q) {
  __shared__ __align__(16) double pool[POOL];
  __shared__ double pivots[NB];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_PANEL + q, it)) return;
  const DirectFront F = a.fronts[it.front];
  if (it.j < 0)
    scale_tile(a, F, q, it.i, pool, pivots);
  else
    update_tile(a, F, q - 1, it.i, it.j, pool);
}

// A tile of a front's assembled columns in the making: K's blocks and the children's Schur
// complements, in LDS with rows of LDN, zero outside.  Tiles lie on the front's diagonal or below.
struct Assembly {
  DirectRows R;
  int c0, nc;
  int e0, e1;             // K's entries
  double* T;              // NB x LDN
};

// Up to ALL of K's blocks of a tile, two values of each of AT_ONCE a thread: all of a thread's loads
// are in flight together (one block after the other took 1.5 us each).
struct KBlocks {
  static constexpr int AT_ONCE = 4, BLOCKS = TPB / 18, ALL = AT_ONCE * BLOCKS;
  DirectEntry en[AT_ONCE];
  double2 x[AT_ONCE];
  __device__ __forceinline__ void entries(const DirectArgs& a, int e0, int e1) {
    const int b = (64 * wave_id() + lane_here()) / 18;
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
      const int e = e0 + b + u * BLOCKS;
      en[u].rc = -1;
      if (b < BLOCKS && e < e1) en[u] = a.entries[e];
    }
  }
  __device__ __forceinline__ void values(const DirectArgs& a) {
    const int q = 2 * ((64 * wave_id() + lane_here()) % 18);
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u)
      if (en[u].rc >= 0)
        x[u] = *reinterpret_cast<const double2*>(a.K + 36 * (int64_t)en[u].slot + q);
  }
  // block (row, col) of the front is the transpose of K's (col, row); every value has one place
  __device__ __forceinline__ void put(const Assembly& A) const {
    const int q = 2 * ((64 * wave_id() + lane_here()) % 18), cb = q / 6, ca = q - 6 * cb;
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
      if (en[u].rc < 0) continue;
      const int r = (en[u].rc >> 16) - DIRECT_EDGE + ca, c = (en[u].rc & 0xffff) - DIRECT_EDGE + cb;
      if (c < 0 || c >= A.nc) continue;
      if (r >= 0 && r < A.R.n) A.T[r * LDN + c] = x[u].x;
      if (r + 1 >= 0 && r + 1 < A.R.n) A.T[(r + 1) * LDN + c] = x[u].y;
    }
  }
};

// A tile's entries a thread holds: column lane, rows wave + TILE_STEP u.
constexpr int TILE_STEP = TPB / 64, TILE_PER = NB / TILE_STEP;
static_assert(NB == 64, "a wave takes a row, and a lane of it knows the map of a row");

// The children's part of a tile.  A lane's column is the lower index in the children as well
// (boundaries keep the order of the parent), so that a wave reads along a row of their triangles:
// a scalar base, and one offset a lane for all rows.  A tile on the diagonal is read in its lower
// half and mirrored.  All of a thread's loads are in flight together from load to add; where a
// column is not wanted, they read the row's first entry.
struct ChildValues {
  int row[2], col[2];            // DOF row lane, column lane of the tile in the children, or -1
  double v[2][TILE_PER];
  __device__ __forceinline__ void maps(const DirectArgs& a, const DirectFront& F,
                                       const Assembly& A) {
    const int lane = lane_here(), cnt = (F.ns6 + F.nb6) / 6;
    const int r = A.R.r0 + lane, c = A.c0 + lane;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int32_t* __restrict__ map = a.maps + F.map_off + k * cnt;
      row[k] = lane < A.R.n ? map[r / 6] : -1;
      col[k] = lane < A.nc ? map[c / 6] : -1;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      row[k] = row[k] < 0 ? -1 : 6 * row[k] + r % 6;
      col[k] = col[k] < 0 ? -1 : 6 * col[k] + c % 6;
    }
  }
  __device__ __forceinline__ void load(const DirectArgs& a, const DirectFront& F,
                                       const Assembly& A) {
    const int lane = lane_here(), wave = wave_id();
    const int last = A.c0 == A.R.r0 ? 0 : NB;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const double* __restrict__ U = a.u + F.child_u[k];
      const unsigned at = col[k] < 0 ? 0u : 8u * (unsigned)col[k];
#pragma unroll
      for (int u = 0; u < TILE_PER; ++u) {
        const int r = __builtin_amdgcn_readlane(row[k], wave + TILE_STEP * u);
        v[k][u] = 0.0;
        if (r >= 0) {
          const char* line = reinterpret_cast<const char*>(U + direct_tri(r));
          const bool low = lane <= wave + TILE_STEP * u + last;
          v[k][u] = *reinterpret_cast<const double*>(line + (low ? at : 0u));
        }
      }
    }
  }
  // into the tile, and into the front's assembled columns where out
  __device__ __forceinline__ void add(const DirectArgs& a, const DirectFront& F, const Assembly& A,
                                      bool leaf, bool out) const {
    const int lane = lane_here(), wave = wave_id();
    const bool diagonal = A.c0 == A.R.r0;
    double* __restrict__ p = a.f0 + F.work_off + (int64_t)(A.R.r0 + wave) * F.ns6 + A.c0 + lane;
    double* __restrict__ q = a.f0 + F.work_off + (int64_t)(A.c0 + lane) * F.ns6 + A.R.r0 + wave;
    double x[TILE_PER];
#pragma unroll
    for (int u = 0; u < TILE_PER; ++u) x[u] = A.T[(wave + TILE_STEP * u) * LDN + lane];
#pragma unroll
    for (int u = 0; u < TILE_PER; ++u) {
      const int r = wave + TILE_STEP * u;
      if (!diagonal || lane <= r) {
        if (!leaf) {
          x[u] += (col[0] >= 0 ? v[0][u] : 0.0) + (col[1] >= 0 ? v[1][u] : 0.0);
          A.T[r * LDN + lane] = x[u];
          if (diagonal) A.T[lane * LDN + r] = x[u];
        }
        if (out && lane < A.nc && r < A.R.n) {
          *p = x[u];
          if (diagonal) *q = x[u];
        }
      }
      p += TILE_STEP * F.ns6;
      q += TILE_STEP;
    }
  }
};

// A tile's transpose into the other half of the front's own columns.
__device__ __forceinline__ void store_mirror(const DirectArgs& a, const DirectFront& F,
                                             const Assembly& A) {
  if (A.c0 == A.R.r0 || A.R.r0 >= F.ns6) return;
  const int lane = lane_here(), wave = wave_id();
  double* __restrict__ p = a.f0 + F.work_off + (int64_t)(A.c0 + wave) * F.ns6 + A.R.r0 + lane;
#pragma unroll
  for (int u = 0; u < TILE_PER; ++u) {
    const int c = wave + TILE_STEP * u;
    if (lane < A.R.n && c < A.nc) *p = A.T[lane * LDN + c];
    p += TILE_STEP * F.ns6;
  }
}

// Assembles N tiles in LDS and, where out, into the front's columns.  What waits for memory is on
// its way for all tiles at once: K's entries and the maps, then K's blocks and the children's
// values.  The workgroup enters with T free.
template <int N>
__device__ __forceinline__ void assemble(const DirectArgs& a, const DirectFront& F, bool leaf,
                                         const Assembly (&A)[N], const bool (&out)[N]) {
  KBlocks kb[N];
  ChildValues cv[N];
  const int lane = lane_here(), wave = wave_id();
#pragma unroll
  for (int k = 0; k < N; ++k) kb[k].entries(a, A[k].e0, A[k].e1);
  if (!leaf) {
#pragma unroll
    for (int k = 0; k < N; ++k) cv[k].maps(a, F, A[k]);
#pragma unroll
    for (int k = 0; k < N; ++k)     // here, not in front of each child's loads
      asm volatile("" : "+v"(cv[k].row[0]), "+v"(cv[k].row[1]), "+v"(cv[k].col[0]),
                        "+v"(cv[k].col[1]));
  }
#pragma unroll
  for (int k = 0; k < N; ++k) {
    double* T = A[k].T + wave * LDN + lane;
#pragma unroll
    for (int u = 0; u < TILE_PER; ++u) T[u * TILE_STEP * LDN] = 0.0;
  }
#pragma unroll
  for (int k = 0; k < N; ++k) kb[k].values(a);
  if (!leaf) {
#pragma unroll
    for (int k = 0; k < N; ++k) cv[k].load(a, F, A[k]);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    kb[k].put(A[k]);
    for (int e = A[k].e0 + KBlocks::ALL; e < A[k].e1; e += KBlocks::ALL) {
      kb[k].entries(a, e, A[k].e1);
      kb[k].values(a);
      kb[k].put(A[k]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) cv[k].add(a, F, A[k], leaf, out[k]);
  __syncthreads();
}

// Step 0 of a level's panels.  Items with j >= 0 assemble tile (i, j) of the front's columns.  The
// others assemble the first column of tiles, -j row tiles from i on, and scale panel 0: the pivot
// block, which each item assembles and inverts for itself, and F_I0 D^-1; the only panel of a front
// goes straight into the factor.
//
// 21 to 25 us on a level with few fronts: 9 in the assembly (four dependent loads, then up to 128 KB
// of the children's values through one CU), 8.3 in the inversion, 2.7 in the product.  A launch that
// assembled into memory and one that read it back took 26 to 28, and on a 300 x 300 shell's levels
// 3.0 ms against 1.6.  The kernel must not use scratch memory: with 400 bytes of it a launch took 10
// us longer.
__global__ void __launch_bounds__(TPB, 2)
k_front_first(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ __align__(16) double T0[NB * LDN];
  __shared__ __align__(16) double T1[NB * LDN];
  __shared__ double pivots[NB];
  static_assert(SWEEP_LDS <= NB * LDN, "the sweep's panel fits a tile");
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_PANEL, it)) return;
  const DirectFront F = a.fronts[it.front];
  const bool leaf = F.child[0] < 0 && F.child[1] < 0;
  int i = it.i;
  if (it.j >= 0) {
    const int c0 = it.j * NB;
    const Assembly tile{direct_rows(F, i), c0, F.ns6 - c0 < NB ? F.ns6 - c0 : NB, it.e0, it.e1, T1};
    assemble<1>(a, F, leaf, {tile}, {true});
    store_mirror(a, F, tile);
    return;
  }
  const int nb = F.ns6 < NB ? F.ns6 : NB;
  const bool only = F.np == 1;      // then only the boundary rows are read again, by the Schur step
  const int64_t ldo = only ? F.ns6 : NB;
  const int end = i - it.j;
  const Assembly pivot{direct_rows(F, 0), 0, nb, F.e0, F.e1, T0};
  if (i == 0) {
    assemble<1>(a, F, leaf, {pivot}, {!only});
  } else {
    const Assembly tile{direct_rows(F, i), 0, nb, it.e0, it.e1, T1};
    assemble<2>(a, F, leaf, {pivot, tile}, {false, true});
    store_mirror(a, F, tile);
  }
  {
    d4 d[2][2];
    const int lane = lane_here(), wave = wave_id();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 32 * (wave >> 1) + 16 * u + (lane >> 4) + 4 * v;
          const int c = 32 * (wave & 1) + 16 * w + (lane & 15);
          d[u][w][v] = r < nb && c < nb ? T0[r * LDN + c] : (r == c ? 1.0 : 0.0);
        }
    __syncthreads();
    sweep(d, nb, T0, pivots);
    each_acc(d, [&](int r, int c, double v) { T0[r * LDN + c] = -v; });
    if (i == 0) {
      check_pivots(a, F, 0, nb, pivots);
      double* __restrict__ out = only ? a.fact + F.fact_off : scaled(a, F, 0, 0);
      each_acc(d, [&](int r, int c, double v) {
        if (r < nb && c < nb) out[(int64_t)r * ldo + c] = only ? v : -v;
      });
    }
  }
  __syncthreads();
  for (bool first_row = true; i < end; ++i, first_row = false) {
    if (i == 0) continue;
    const DirectRows R = direct_rows(F, i);
    if (!first_row) {
      const Assembly tile{R, 0, nb, a.tile_end[F.tile_off + i - 1], a.tile_end[F.tile_off + i], T1};
      __syncthreads();
      assemble<1>(a, F, leaf, {tile}, {true});
      store_mirror(a, F, tile);
    }
    double* __restrict__ out =
        only ? a.fact + F.fact_off + (int64_t)R.r0 * F.ns6 : scaled(a, F, 0, i);
    d4 acc[2][2];
    clear(acc);
    if (nb == NB) {
      mma_tile(T1, LDN, T0, LDN, KC, acc);
      mma_tile(T1 + KC, LDN, T0 + KC, LDN, KC, acc);
    } else {
      mma_tile(T1, LDN, T0, LDN, (nb + 3) & ~3, acc);
    }
    each_acc(acc, [&](int r, int c, double v) {
      if (r < R.n && c < nb) out[(int64_t)r * ldo + c] = v;
    });
  }
}

// Tile (i, j) of a front's boundary rows: G = F_BS W, from the own rows, which hold -W by then.
// One product over all own columns, where the panel steps would read and write each boundary tile
// once a panel: with 1806 boundary and 900 own DOFs, four fronts, 15 panel steps took 60 us each,
// 28 without the boundary rows, which take 286 here (48 TFLOP/s); 300 x 300 shell: 12.7 -> 11.3 ms.
__global__ void __launch_bounds__(TPB)
k_front_gain(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ double as[NB * LDK];
  __shared__ double bs[NB * LDK];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_GAIN, it)) return;
  const DirectFront F = a.fronts[it.front];
  const DirectRows R = direct_rows(F, it.i);
  const int c0 = it.j * NB, nc = F.ns6 - c0 < NB ? F.ns6 - c0 : NB;
  d4 acc[2][2];
  clear(acc);
  product(a.f0 + F.work_off + (int64_t)R.r0 * F.ns6, F.ns6, R.n,
          a.fact + F.fact_off + (int64_t)c0 * F.ns6, F.ns6, nc, F.ns6, as, bs, acc);
  double* __restrict__ out = a.fact + F.fact_off + (int64_t)R.r0 * F.ns6 + c0;
  each_acc(acc, [&](int r, int c, double v) {
    if (r < R.n && c < nc) out[(int64_t)r * F.ns6 + c] = -v;
  });
}

// Tile (i, j), j <= i, of a front's Schur complement: the children's minus G F_BS^T.  With several
// panels and no gain step that product is the sum over the panels but the last of G before it times
// F_BS, plus the last panel's scaled columns times what they were before (both are G F_BS^T), so
// that the columns' update with the last panel is other items of the same launch: one of 9 us less
// a level.
//
// 12 to 15 us on a level with few fronts; 50 TFLOP/s on wide fronts (1806 boundary and 900 own DOFs),
// half of that on a 300 x 300 shell's lower levels, bound by the latency of their short products.
__global__ void __launch_bounds__(TPB)
k_front_schur(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ double pool[2 * NB * LDK];
  double* as = pool;
  double* bs = pool + NB * LDK;
  __shared__ int mr[2][NB], mc[2][NB];     // 6 * position in the child's boundary, or -1
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_SCHUR, it)) return;
  const DirectFront F = a.fronts[it.front];
  if (it.e0) {
    update_tile(a, F, F.np - 1, it.i, it.j, pool);
    return;
  }
  const int ns = F.ns6 / 6, cnt = ns + F.nb6 / 6;
  const int r0 = it.i * NB, c0 = it.j * NB;
  const int nr = F.nb6 - r0 < NB ? F.nb6 - r0 : NB, nc = F.nb6 - c0 < NB ? F.nb6 - c0 : NB;
  {
    const int t = threadIdx.x, k = t >> 7, q = t & 63;
    const int row = ((t >> 6) & 1) ? c0 + q : r0 + q;
    int m = -1;
    if (row < F.nb6) {
      m = a.maps[F.map_off + k * cnt + ns + row / 6];
      if (m >= 0) m = 6 * m + row % 6;
    }
    if ((t >> 6) & 1)
      mc[k][q] = m;
    else
      mr[k][q] = m;
  }
  // without a gain step the boundary rows as they are before the last panel, that panel apart
  const bool before = F.np > 1 && !F.gain;
  const int split = before ? (F.np - 1) * NB : F.ns6;
  const double* __restrict__ G =
      (before ? sweep_src(a, F, F.np - 1) : a.fact + F.fact_off) + (int64_t)(F.ns6 + r0) * F.ns6;
  const double* __restrict__ B = a.f0 + F.work_off + (int64_t)(F.ns6 + c0) * F.ns6;
  const ChildU u0{a.u + F.child_u[0]}, u1{a.u + F.child_u[1]};
  d4 acc[2][2], sum[2][2];
  clear(acc);
  clear(sum);
  __syncthreads();
  if (F.child[0] >= 0 || F.child[1] >= 0) {   // on their way while the product runs
    const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 32 * (wave >> 1) + 16 * u + (lane >> 4) + 4 * v;
          const int c = 32 * (wave & 1) + 16 * w + (lane & 15);
          sum[u][w][v] = u0.at(mr[0][r], mc[0][c]) + u1.at(mr[1][r], mc[1][c]);
        }
  }
  if (before)
    product(G, F.ns6, nr, B, F.ns6, nc, F.ns6, as, bs, acc, split,
            scaled(a, F, F.np - 1, F.np + it.i), unscaled(a, F, F.np + it.j));
  else
    product(G, F.ns6, nr, B, F.ns6, nc, F.ns6, as, bs, acc);
  double* __restrict__ U = a.u + F.u_off;
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int w = 0; w < 2; ++w) sum[u][w] -= acc[u][w];
  each_acc(sum, [&](int r, int c, double v) {
    if (r < nr && c0 + c <= r0 + r) U[direct_tri(r0 + r) + c0 + c] = v;
  });
}

// Up: b_S (every item of the front for itself, in LDS) and rows [i, e0) of v_B, 16 a pass, 16 lanes
// a row.  A row's first 128 columns are on their way before b_S is there, those of the next pass
// before this one's sum is taken.
//
// Bound by the factor's bytes on levels with many fronts, by latency on the others.  Rows of 64
// lanes left most of them idle on the lowest levels (35 own DOFs on average), and LDS for the
// largest front let three workgroups on a CU: for a 300 x 300 shell (1.05 GB of it) 1.05 ms then,
// 0.36 now; 6.4 us a level of a 60 x 60 one then, 4.7 now.
__global__ void __launch_bounds__(TPB)
k_front_forward(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  extern __shared__ __align__(16) double b[];
  static_assert(FWD_LANES == 16, "a row's sum is taken over a DPP row");
  constexpr int AT_ONCE = 4, COLS = 2 * FWD_LANES;
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_FWD, it)) return;
  const DirectFront F = a.fronts[it.front];
  const int ns = F.ns6 / 6, cnt = ns + F.nb6 / 6;
  const int32_t* __restrict__ m0 = a.maps + F.map_off;
  const int32_t* __restrict__ m1 = m0 + cnt;
  const double* v0 = F.child[0] >= 0 ? a.v + a.fronts[F.child[0]].v_off : nullptr;
  const double* v1 = F.child[1] >= 0 ? a.v + a.fronts[F.child[1]].v_off : nullptr;
  const int l = threadIdx.x % FWD_LANES, r0 = it.i + (int)threadIdx.x / FWD_LANES;
  const double* __restrict__ G = a.fact + F.fact_off + (int64_t)F.ns6 * F.ns6;
  double2 g[AT_ONCE];
  double child = 0.0;                   // lanes 0 and 1: the children's part of the row
  auto fetch = [&](int row, int c0) {
    const double* __restrict__ p = G + (int64_t)row * F.ns6;
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) {
      const int c = c0 + 2 * l + COLS * k;
      g[k] = double2{0.0, 0.0};
      if (row < it.e0 && c < F.ns6) g[k] = *reinterpret_cast<const double2*>(p + c);
    }
  };
  auto fetch_child = [&](int row) {
    child = 0.0;
    if (l < 2 && row < it.e0) {
      const int m = (l ? m1 : m0)[ns + row / 6];
      if (m >= 0) child = (l ? v1 : v0)[6 * m + row % 6];
    }
  };
  fetch(r0, 0);
  for (int c = threadIdx.x; c < F.ns6; c += TPB) {
    const int q = c / 6, d = c - 6 * q;
    const int p0 = m0[q], p1 = m1[q];
    const double v = a.rhs[6 * (int64_t)a.nodes[F.nodes_off + q] + d] +
                     ((p0 >= 0 ? v0[6 * p0 + d] : 0.0) + (p1 >= 0 ? v1[6 * p1 + d] : 0.0));
    b[c] = v;
    if (it.i == 0) a.b[F.b_off + c] = v;
  }
  fetch_child(r0);
  __syncthreads();
  for (int base = it.i; base < it.e0; base += DIRECT_FWD_ROWS) {
    const int row = r0 + base - it.i;
    double s = -child;
    for (int c0 = 0; c0 < F.ns6; c0 += COLS * AT_ONCE) {
      if (c0) fetch(row, c0);
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) {
        const int c = c0 + 2 * l + COLS * k;
        if (c < F.ns6) {
          const double2 bv = *reinterpret_cast<const double2*>(b + c);
          s += g[k].x * bv.x + g[k].y * bv.y;
        }
      }
    }
    if (base + DIRECT_FWD_ROWS < it.e0) {
      fetch(row + DIRECT_FWD_ROWS, 0);
      fetch_child(row + DIRECT_FWD_ROWS);
    }
    s = row_sum(s);
    if (l == 0 && row < it.e0) a.v[F.v_off + row] = -s;
  }
}

// Down: 32 columns of x_S = -(panel^T [b_S; x_B]), the panel's rows dealt to 16 groups of lanes, the
// first 8 of each on their way while the vector is gathered: 5.9 -> 5.4 us a level of a 60 x 60 shell.
__global__ void __launch_bounds__(BWD_TPB)
k_front_backward(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ double y[BWD_CHUNK];
  __shared__ double part[BWD_GROUPS][DIRECT_BWD_COLS + 1];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_BWD, it)) return;
  const DirectFront F = a.fronts[it.front];
  const int rows = F.ns6 + F.nb6;
  const int lc = threadIdx.x % DIRECT_BWD_COLS, g = threadIdx.x / DIRECT_BWD_COLS;
  const int c = it.i * DIRECT_BWD_COLS + lc;
  const int cl = c < F.ns6 ? c : F.ns6 - 1;
  const double* __restrict__ P = a.fact + F.fact_off + cl;
  double s = 0.0;
  constexpr int AT_ONCE = 8;
  double v[AT_ONCE];
  auto fetch = [&](int r, int end) {      // past the end, the last row
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
      const int k = r + u * BWD_GROUPS;
      v[u] = P[(int64_t)(k < end ? k : end - 1) * F.ns6];
    }
  };
  for (int base = 0; base < rows; base += BWD_CHUNK) {
    const int n = rows - base < BWD_CHUNK ? rows - base : BWD_CHUNK;
    fetch(base + g, base + n);          // on its way while y is gathered
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += BWD_TPB) {
      const int r = base + k, q = r / 6;
      y[k] = r < F.ns6 ? a.b[F.b_off + r]
                       : a.sol[6 * (int64_t)a.nodes[F.nodes_off + q] + r - 6 * q];
    }
    __syncthreads();
    for (int k = g; k < n; k += AT_ONCE * BWD_GROUPS) {
      if (k != g) fetch(base + k, base + n);
#pragma unroll
      for (int u = 0; u < AT_ONCE; ++u) {
        const int r = k + u * BWD_GROUPS;
        s += v[u] * (r < n ? y[r] : 0.0);
      }
    }
  }
  part[g][lc] = s;
  __syncthreads();
  if (g == 0 && c < F.ns6) {
    double x = 0.0;
    for (int k = 0; k < BWD_GROUPS; ++k) x += part[k][lc];
    const int q = c / 6;
    a.sol[6 * (int64_t)a.nodes[F.nodes_off + q] + c - 6 * q] = -x;
  }
}

__global__ void k_direct_clear(DirectArgs a, const DirectArgs* __restrict__ probs, int n) {
  const int i = (int)threadIdx.x + (int)(blockIdx.x * blockDim.x);
  if (i < n) *(probs ? probs[i].flag : a.flag) = 0u;
}

// The problems of one launch: a single one by value, or n with their arguments on the device.
struct Launch {
  const DirectPlan* const* plans;
  int n;
  const DirectArgs* one;       // n == 1 and probs == nullptr
  const DirectArgs* probs;
  hipStream_t s;

  int levels() const {
    int h = 0;
    for (int i = 0; i < n; ++i) h = plans[i]->levels() > h ? plans[i]->levels() : h;
    return h;
  }
  int panels(int level) const {
    int q = 0;
    for (int i = 0; i < n; ++i)
      if (level < plans[i]->levels() && plans[i]->level_np[level] > q)
        q = plans[i]->level_np[level];
    return q;
  }
  size_t own(int level) const {
    int c = 0;
    for (int i = 0; i < n; ++i)
      if (level < plans[i]->levels() && plans[i]->level_own[level] > c)
        c = plans[i]->level_own[level];
    return sizeof(double) * (size_t)c;
  }
  // launch(grid, first item) for a step of a level, if any problem has items there
  template <class Fn>
  hipError_t step(int level, int step, Fn launch) const {
    int cnt = 0, first = 0;
    for (int i = 0; i < n; ++i) {
      const DirectPlan& pl = *plans[i];
      if (level >= pl.levels() || step - STEP_PANEL > pl.level_np[level]) continue;
      const DirectRange r = pl.steps[pl.level_off[level] + step];
      cnt = r.cnt > cnt ? r.cnt : cnt;
      first = r.off;
    }
    if (cnt == 0) return hipSuccess;
    launch(dim3((unsigned)cnt, (unsigned)n), first);
    return hipGetLastError();
  }
};

}  // namespace

#define SSO_TRY(x)                 \
  do {                             \
    hipError_t e_ = (x);           \
    if (e_ != hipSuccess) return e_; \
  } while (0)

static hipError_t factor(const Launch& L) {
  const DirectArgs a = L.one ? *L.one : DirectArgs{};
  for (int h = 0; h < L.levels(); ++h) {
    SSO_TRY(L.step(h, STEP_PANEL, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_first, g, dim3(TPB), 0, L.s, a, L.probs, off, h);
    }));
    for (int q = 1; q <= L.panels(h); ++q)
      SSO_TRY(L.step(h, STEP_PANEL + q, [&](dim3 g, int off) {
        hipLaunchKernelGGL(k_front_panel, g, dim3(TPB), 0, L.s, a, L.probs, off, h, q);
      }));
    SSO_TRY(L.step(h, STEP_GAIN, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_gain, g, dim3(TPB), 0, L.s, a, L.probs, off, h);
    }));
    SSO_TRY(L.step(h, STEP_SCHUR, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_schur, g, dim3(TPB), 0, L.s, a, L.probs, off, h);
    }));
  }
  return hipSuccess;
}

static hipError_t substitute(const Launch& L) {
  const DirectArgs a = L.one ? *L.one : DirectArgs{};
  for (int h = 0; h < L.levels(); ++h)
    SSO_TRY(L.step(h, STEP_FWD, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_forward, g, dim3(TPB), L.own(h), L.s, a, L.probs, off, h);
    }));
  for (int h = L.levels() - 1; h >= 0; --h)
    SSO_TRY(L.step(h, STEP_BWD, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_backward, g, dim3(BWD_TPB), 0, L.s, a, L.probs, off, h);
    }));
  return hipSuccess;
}

hipError_t launch_direct_clear(const DirectArgs& a, hipStream_t s) {
  const DirectArgs* none = nullptr;
  hipLaunchKernelGGL(k_direct_clear, dim3(1), dim3(64), 0, s, a, none, 1);
  return hipGetLastError();
}

hipError_t launch_direct_factor(const DirectPlan& pl, const DirectArgs& a, hipStream_t s) {
  const DirectPlan* p = &pl;
  return factor(Launch{&p, 1, &a, nullptr, s});
}

hipError_t launch_direct_solve(const DirectPlan& pl, const DirectArgs& a, hipStream_t s) {
  const DirectPlan* p = &pl;
  return substitute(Launch{&p, 1, &a, nullptr, s});
}

hipError_t direct_batch_reserve(int n, DirectBatch& db, hipStream_t s) {
  if (n > db.cap) {   // nothing is pending: the last launch was waited for
    dev_free(db.d, s);
    dev_free(db.d_res, s);
    dev_free(db.d_out, s);
    db.d = nullptr;
    db.d_res = nullptr;
    db.d_out = nullptr;
    db.cap = 0;
    SSO_TRY(dev_alloc_scratch(&db.d, 2 * n, s));
    SSO_TRY(dev_alloc_scratch(&db.d_res, 2 * n, s));
    SSO_TRY(dev_alloc_scratch(&db.d_out, 6 * n, s));
    db.cap = 2 * n;
  }
  if (!db.ev) SSO_TRY(hipEventCreateWithFlags(&db.ev, hipEventDisableTiming));
  db.h.resize(n);
  db.h_res.resize(n);
  db.plans.resize(n);
  db.out.resize(3 * n);
  return hipSuccess;
}

hipError_t direct_batch_launch(const std::vector<DirectJob>& jobs, DirectBatch& db,
                               hipStream_t s) {
  const int n = (int)jobs.size();
  SSO_TRY(direct_batch_reserve(n, db, s));
  int nf = 0;
  for (int i = 0; i < n; ++i) {
    db.h[i] = jobs[i].a;
    db.h_res[i] = jobs[i].residual;
    db.plans[i] = jobs[i].plan;
    if (jobs[i].factor) nf = i + 1;
  }
  SSO_TRY(hipMemcpyAsync(db.d, db.h.data(), sizeof(DirectArgs) * n, hipMemcpyHostToDevice, s));
  SSO_TRY(hipMemcpyAsync(db.d_res, db.h_res.data(), sizeof(ResidualJob) * n,
                         hipMemcpyHostToDevice, s));
  if (nf > 0) {
    hipLaunchKernelGGL(k_direct_clear, dim3((unsigned)((nf + 63) / 64)), dim3(64), 0, s,
                       DirectArgs{}, db.d, nf);
    SSO_TRY(hipGetLastError());
    SSO_TRY(factor(Launch{db.plans.data(), nf, nullptr, db.d, s}));
  }
  SSO_TRY(substitute(Launch{db.plans.data(), n, nullptr, db.d, s}));
  SSO_TRY(launch_residuals(db.h_res, db.d_res, db.d_out, s));
  return hipEventRecord(db.ev, s);
}

hipError_t direct_batch_wait(DirectBatch& db, hipStream_t s) {
  SSO_TRY(hipEventSynchronize(db.ev));
  SSO_TRY(hipMemcpyAsync(db.out.data(), db.d_out, sizeof(double) * db.out.size(),
                         hipMemcpyDeviceToHost, s));
  return hipStreamSynchronize(s);
}

void direct_batch_free(DirectBatch& db, hipStream_t s) {
  if (db.ev) {
    (void)hipEventSynchronize(db.ev);
    (void)hipEventDestroy(db.ev);
  }
  dev_free(db.d, s);
  dev_free(db.d_res, s);
  dev_free(db.d_out, s);
  db = DirectBatch();
}

}  // namespace sso
