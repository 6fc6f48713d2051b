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
// after which the own rows hold -W and the boundary rows G.  Sweeps alternate between two copies
// of the panel (k_front_scale forms F_IJ D^-1, k_front_update the rest), so no work item reads
// what another one of the same launch writes.  The products run on the matrix cores
// (v_mfma_f64_16x16x4_f64) from LDS tiles.  All fronts of one level share the launches; the items
// of a launch come from the plan, so a front's arithmetic does not depend on what else is in the
// launch.  No atomics: every entry has one writer and a fixed order of additions.
#include <cmath>

#include "sso_internal.h"

namespace sso {
namespace {

constexpr int NB = DIRECT_NB;
constexpr int TPB = 256;
constexpr int KC = 32;                // depth of an LDS tile
constexpr int LDK = KC + 1;           // its row length: odd, so that 16 rows spread over the banks
constexpr int LDN = NB + 1;
constexpr int ASM_R = 6 * DIRECT_ASM_ROWS, ASM_C = 6 * DIRECT_ASM_COLS;
constexpr int BWD_TPB = 512;
constexpr int BWD_GROUPS = BWD_TPB / DIRECT_BWD_COLS;
constexpr int BWD_CHUNK = 2048;       // rows of the vector staged at a time
// A pivot below this share of K's diagonal entry means that K is singular to working precision
// (rounding leaves some 1e-15 of it in place of a zero pivot); the solve then goes back to PCG.
constexpr double PIVOT_MIN = 1e-13;

typedef double d4 __attribute__((ext_vector_type(4)));

// The item of this workgroup, or false past the end of the problem's list.  probs == nullptr: one
// problem, given by value with its list's offset; else problem blockIdx.y, whose list is looked up.
__device__ __forceinline__ bool take_item(DirectArgs& a, const DirectArgs* __restrict__ probs,
                                          int first, int level, int step, DirectItem& it) {
  if (probs) {
    a = probs[blockIdx.y];
    if (level >= a.n_levels) return false;
    if (step >= STEP_PANEL && (step - STEP_PANEL) / 2 >= a.level_np[level]) return false;
    const DirectRange r = a.steps[a.level_off[level] + step];
    if ((int)blockIdx.x >= r.cnt) return false;
    first = r.off;
  }
  it = a.items[first + (int)blockIdx.x];
  return true;
}

// Entry (r, c) of the Schur complements of a front's children at two nodes given by their
// positions in the children's boundaries (-1: not there), components ca and cb.  A child's U
// holds its lower triangle; the maps ascend, so both children keep the order of the rows.
struct ChildU {
  const double* u;
  int ld;
};
__device__ __forceinline__ double child_entry(const ChildU& u, int mr, int mc, int ca, int cb) {
  if ((mr | mc) < 0) return 0.0;
  const int r = 6 * mr + ca, c = 6 * mc + cb;
  const int hi = r > c ? r : c, lo = r > c ? c : r;
  return u.u[(int64_t)hi * u.ld + lo];
}
__device__ __forceinline__ ChildU child_of(const DirectArgs& a, int f) {
  ChildU u{nullptr, 0};
  if (f >= 0) {
    u.u = a.u + a.fronts[f].u_off;
    u.ld = a.fronts[f].nb6;
  }
  return u;
}

// A front's columns: children's Schur complements and K's blocks, a tile of 8 x 16 nodes in LDS.
__global__ void __launch_bounds__(TPB)
k_front_assemble(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ double tile[ASM_R * ASM_C];
  __shared__ int mr[2][DIRECT_ASM_ROWS], mc[2][DIRECT_ASM_COLS];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_ASM, it)) return;
  const DirectFront F = a.fronts[it.front];
  const int ns = F.ns6 / 6, cnt = ns + F.nb6 / 6;
  const int rn0 = it.i * DIRECT_ASM_ROWS, cn0 = it.j * DIRECT_ASM_COLS;
  const int t = threadIdx.x;
  if (t < 2 * DIRECT_ASM_ROWS) {
    const int k = t / DIRECT_ASM_ROWS, r = t % DIRECT_ASM_ROWS;
    mr[k][r] = rn0 + r < cnt ? a.maps[F.map_off + k * cnt + rn0 + r] : -1;
  } else if (t >= 64 && t < 64 + 2 * DIRECT_ASM_COLS) {
    const int k = (t - 64) / DIRECT_ASM_COLS, c = (t - 64) % DIRECT_ASM_COLS;
    mc[k][c] = cn0 + c < ns ? a.maps[F.map_off + k * cnt + cn0 + c] : -1;
  }
  const ChildU u0 = child_of(a, F.child[0]), u1 = child_of(a, F.child[1]);
  __syncthreads();
  for (int e = t; e < ASM_R * ASM_C; e += TPB) {
    const int r = e / ASM_C, c = e - r * ASM_C;
    const int rn = r / 6, cn = c / 6;
    tile[e] = child_entry(u0, mr[0][rn], mc[0][cn], r - 6 * rn, c - 6 * cn) +
              child_entry(u1, mr[1][rn], mc[1][cn], r - 6 * rn, c - 6 * cn);
  }
  __syncthreads();
  // K's blocks: block (row, col) of the front is the transpose of K's (col, row)
  for (int e = t; e < 36 * (it.e1 - it.e0); e += TPB) {
    const int k = e / 36, q = e - 36 * k;
    const DirectEntry en = a.entries[it.e0 + k];
    const int cb = q / 6, ca = q - 6 * cb;       // K entry (cb, ca) of block (col node, row node)
    tile[(6 * (en.rc >> 16) + ca) * ASM_C + 6 * (en.rc & 0xffff) + cb] +=
        a.K[36 * (int64_t)en.slot + q];
  }
  __syncthreads();
  double* out = a.f0 + F.work_off;
  const int rows = F.ns6 + F.nb6 - 6 * rn0, cols = F.ns6 - 6 * cn0;
  for (int e = t; e < ASM_R * ASM_C; e += TPB) {
    const int r = e / ASM_C, c = e - r * ASM_C;
    if (r < rows && c < cols) out[(int64_t)(6 * rn0 + r) * F.ns6 + 6 * cn0 + c] = tile[e];
  }
}

// Where a front's sweep p reads and writes its columns: the last one writes the factor, the ones
// before alternate, the first reads the assembled front.
__device__ __forceinline__ double* sweep_dst(const DirectArgs& a, const DirectFront& F, int p) {
  return ((F.np - 1 - p) & 1) == 0 ? a.fact + F.fact_off : a.x1 + F.again_off;
}
__device__ __forceinline__ const double* sweep_src(const DirectArgs& a, const DirectFront& F,
                                                   int p) {
  return p == 0 ? a.f0 + F.work_off : sweep_dst(a, F, p - 1);
}

// Rows of row tile i of a front (own rows first, boundary rows in tiles of their own).
struct RowTile {
  int r0, n;
};
__device__ __forceinline__ RowTile row_tile(const DirectFront& F, int i) {
  RowTile t;
  if (i < F.np) {
    t.r0 = i * NB;
    t.n = F.ns6 - t.r0;
  } else {
    t.r0 = F.ns6 + (i - F.np) * NB;
    t.n = F.ns6 + F.nb6 - t.r0;
  }
  if (t.n > NB) t.n = NB;
  return t;
}

// A tile of up to 64 rows x KC columns of a row-major array into LDS, zero outside.
__device__ __forceinline__ void load_tile(const double* __restrict__ src, int64_t ld, int rows,
                                          int k0, int kn, double* dst) {
  // 16-byte loads: rows start at even offsets (every row length is a multiple of 6 or 64)
  for (int e = threadIdx.x; e < NB * KC / 2; e += TPB) {
    const int r = e / (KC / 2), c = 2 * (e - r * (KC / 2));
    double2 v{0.0, 0.0};
    if (r < rows && k0 + c < kn)
      v = *reinterpret_cast<const double2*>(src + (int64_t)r * ld + k0 + c);
    dst[r * LDK + c] = v.x;
    dst[r * LDK + c + 1] = v.y;   // kn is even: a pair lies inside or outside as a whole
  }
}

// acc += A B^T over KC columns of LDS tiles A, B (64 x KC each): the wave's 32 x 32 quadrant as
// 2 x 2 matrix-core tiles.  kn: columns that hold values.
__device__ __forceinline__ void mma_tile(const double* A, int lda, const double* B, int ldb,
                                         int kn, d4 acc[2][2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const double* pa = A + (32 * (wave >> 1) + l16) * lda + kq;
  const double* pb = B + (32 * (wave & 1) + l16) * ldb + kq;
  for (int k = 0; k < kn; k += 4) {
    const double a0 = pa[k], a1 = pa[16 * lda + k];
    const double b0 = pb[k], b1 = pb[16 * ldb + k];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
}

// f(row, column, value) over the wave's accumulators: lane l holds column l % 16 and rows
// l / 16 + 4 v of each 16 x 16 tile.
template <class Fn>
__device__ __forceinline__ void each_acc(const d4 acc[2][2], Fn f) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
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

// Sweep p, first half: D^-1 of the front's pivot block (by every workgroup of the front for
// itself: it costs no more time than one of them doing it first) and F_IJ D^-1 for one row tile.
// D is swept column by column in registers, 4 x 4 entries a thread; a step publishes the pivot
// column through LDS (the matrix stays symmetric, so it is the pivot row as well) and needs one
// barrier, the buffers alternating.
__global__ void __launch_bounds__(TPB)
k_front_scale(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level, int p) {
  __shared__ double ds[NB * LDN];
  __shared__ double as[NB * LDK];
  __shared__ double col[2][NB];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_PANEL + 2 * p, it)) return;
  const DirectFront F = a.fronts[it.front];
  const double* __restrict__ src = sweep_src(a, F, p);
  const int64_t ld = F.ns6;
  const int j0 = p * NB;
  const int nb = F.ns6 - j0 < NB ? F.ns6 - j0 : NB;
  const int t = threadIdx.x, ty = t >> 4, tx = t & 15;
  double d[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = 4 * ty + i, c = 4 * tx + j;
      d[i][j] = r < nb && c < nb ? src[(int64_t)(j0 + r) * ld + j0 + c] : (r == c ? 1.0 : 0.0);
    }
  // the smallest pivot allowed at this thread's diagonal entries
  double least[4] = {0.0, 0.0, 0.0, 0.0};
  if (ty == tx && it.i == p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 4 * ty + i;
      if (r < nb) {
        const int q = (j0 + r) / 6, c = (j0 + r) - 6 * q;
        least[i] = PIVOT_MIN * a.K[36 * (int64_t)a.bdiag[a.nodes[F.nodes_off + q]] + 7 * c];
      }
    }
  }
  bool bad = false;
  const int steps = (nb + 3) / 4;
  for (int k4 = 0; k4 < steps; ++k4) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int k = 4 * k4 + kk;
      double* cb = col[k & 1];
      if (tx == k4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) cb[4 * ty + i] = d[i][kk];
      }
      __syncthreads();
      const double piv = cb[k];
      if (ty == k4 && tx == k4 && !(piv > least[kk])) bad = true;
      const double inv = 1.0 / piv;
      double cr[4], cc[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) cr[i] = cb[4 * ty + i] * inv;
#pragma unroll
      for (int j = 0; j < 4; ++j) cc[j] = cb[4 * tx + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool rk = 4 * ty + i == k, ck = 4 * tx + j == k;
          const double up = d[i][j] - cr[i] * cc[j];
          d[i][j] = rk ? (ck ? -inv : cc[j] * inv) : (ck ? cr[i] : up);
        }
    }
  }
  if (it.i == p && bad) atomicOr(a.flag, 1u);
  const RowTile R = row_tile(F, it.i);
  const bool only = F.np == 1;    // no second half: straight into the factor
  if (it.i == p) {
    double* out = only ? a.fact + F.fact_off : a.w + F.w_off + (int64_t)it.i * NB * NB;
    const int64_t ldo = only ? ld : NB;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 4 * ty + i, c = 4 * tx + j;
        if (r < nb && c < nb) out[(int64_t)r * ldo + c] = only ? d[i][j] : -d[i][j];
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) ds[(4 * ty + i) * LDN + 4 * tx + j] = -d[i][j];
  d4 acc[2][2];
  clear(acc);
  for (int k0 = 0; k0 < nb; k0 += KC) {
    __syncthreads();
    load_tile(src + (int64_t)R.r0 * ld + j0, ld, R.n, k0, nb, as);
    __syncthreads();
    mma_tile(as, LDK, ds + k0, LDN, nb - k0 < KC ? nb - k0 : KC, acc);
  }
  double* out = only ? a.fact + F.fact_off + (int64_t)R.r0 * ld
                     : a.w + F.w_off + (int64_t)it.i * NB * NB;
  const int64_t ldo = only ? ld : NB;
  each_acc(acc, [&](int r, int c, double v) {
    if (r < R.n && c < nb) out[(int64_t)r * ldo + c] = v;
  });
}

// Sweep p, second half: tile (i, j) of the front's columns from one copy to the other.
__global__ void __launch_bounds__(TPB)
k_front_update(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level, int p) {
  __shared__ double as[NB * LDK];
  __shared__ double bs[NB * LDK];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_PANEL + 2 * p + 1, it)) return;
  const DirectFront F = a.fronts[it.front];
  const double* __restrict__ src = sweep_src(a, F, p);
  double* __restrict__ dst = sweep_dst(a, F, p);
  const int64_t ld = F.ns6;
  const int j0 = p * NB;
  const int nb = F.ns6 - j0 < NB ? F.ns6 - j0 : NB;
  const RowTile R = row_tile(F, it.i);
  const int c0 = it.j * NB;
  const int nc = F.ns6 - c0 < NB ? F.ns6 - c0 : NB;
  const double* __restrict__ w = a.w + F.w_off;
  if (it.j == p || it.i == p) {
    // the panel's own column (F_IJ D^-1, -D^-1 on the diagonal) and row (its transpose)
    const double* __restrict__ wi = w + (int64_t)it.i * NB * NB;
    const double* __restrict__ wj = w + (int64_t)it.j * NB * NB;
    for (int e = threadIdx.x; e < NB * NB; e += TPB) {
      const int r = e / NB, c = e - r * NB;
      if (r >= R.n || c >= nc) continue;
      const double v = it.j == p ? (it.i == p ? -wi[r * NB + c] : wi[r * NB + c])
                                 : wj[c * NB + r];
      dst[(int64_t)(R.r0 + r) * ld + c0 + c] = v;
    }
    return;
  }
  d4 acc[2][2];
  clear(acc);
  for (int k0 = 0; k0 < nb; k0 += KC) {
    load_tile(w + (int64_t)it.i * NB * NB, NB, R.n, k0, nb, as);
    load_tile(src + (int64_t)c0 * ld + j0, ld, nc, k0, nb, bs);
    __syncthreads();
    mma_tile(as, LDK, bs, LDK, nb - k0 < KC ? nb - k0 : KC, acc);
    __syncthreads();
  }
  each_acc(acc, [&](int r, int c, double v) {
    if (r < R.n && c < nc) {
      const int64_t q = (int64_t)(R.r0 + r) * ld + c0 + c;
      dst[q] = src[q] - v;
    }
  });
}

// Tile (i, j), j <= i, of a front's Schur complement: the children's minus G F_BS^T.
__global__ void __launch_bounds__(TPB)
k_front_schur(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ double as[NB * LDK];
  __shared__ double bs[NB * LDK];
  __shared__ int mr[2][NB], mc[2][NB];     // 6 * position in the child's boundary, or -1
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_SCHUR, it)) return;
  const DirectFront F = a.fronts[it.front];
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
  const double* __restrict__ G = a.fact + F.fact_off + (int64_t)(F.ns6 + r0) * F.ns6;
  const double* __restrict__ B = a.f0 + F.work_off + (int64_t)(F.ns6 + c0) * F.ns6;
  d4 acc[2][2];
  clear(acc);
  for (int k0 = 0; k0 < F.ns6; k0 += KC) {
    load_tile(G, F.ns6, nr, k0, F.ns6, as);
    load_tile(B, F.ns6, nc, k0, F.ns6, bs);
    __syncthreads();
    mma_tile(as, LDK, bs, LDK, F.ns6 - k0 < KC ? (F.ns6 - k0 + 3) & ~3 : KC, acc);
    __syncthreads();
  }
  if (F.ns6 == 0) __syncthreads();
  const ChildU u0 = child_of(a, F.child[0]), u1 = child_of(a, F.child[1]);
  double* __restrict__ U = a.u + F.u_off;
  each_acc(acc, [&](int r, int c, double v) {
    if (r >= nr || c >= nc) return;
    auto child = [&](const ChildU& u, int ir, int ic) {
      if ((ir | ic) < 0) return 0.0;
      const int hi = ir > ic ? ir : ic, lo = ir > ic ? ic : ir;
      return u.u[(int64_t)hi * u.ld + lo];
    };
    const double s = child(u0, mr[0][r], mc[0][c]) + child(u1, mr[1][r], mc[1][c]);
    U[(int64_t)(r0 + r) * F.nb6 + c0 + c] = s - v;
  });
}

// Up: b_S (every workgroup of the front for itself) and 64 rows of v_B.  A wave takes a row at a
// time, its lanes along the row.
__global__ void __launch_bounds__(TPB)
k_front_forward(DirectArgs a, const DirectArgs* __restrict__ probs, int first, int level) {
  __shared__ __align__(16) double b[DIRECT_MAX_OWN];
  DirectItem it;
  if (!take_item(a, probs, first, level, STEP_FWD, it)) return;
  const DirectFront F = a.fronts[it.front];
  const int ns = F.ns6 / 6, cnt = ns + F.nb6 / 6;
  const int32_t* __restrict__ m0 = a.maps + F.map_off;
  const int32_t* __restrict__ m1 = m0 + cnt;
  const double* v0 = F.child[0] >= 0 ? a.v + a.fronts[F.child[0]].v_off : nullptr;
  const double* v1 = F.child[1] >= 0 ? a.v + a.fronts[F.child[1]].v_off : nullptr;
  auto children = [&](int node, int c) {
    const int p0 = m0[node], p1 = m1[node];
    return (p0 >= 0 ? v0[6 * p0 + c] : 0.0) + (p1 >= 0 ? v1[6 * p1 + c] : 0.0);
  };
  for (int c = threadIdx.x; c < F.ns6; c += TPB) {
    const int q = c / 6, d = c - 6 * q;
    const double v = a.rhs[6 * (int64_t)a.nodes[F.nodes_off + q] + d] + children(q, d);
    b[c] = v;
    if (it.i == 0) a.b[F.b_off + c] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r_end = F.nb6 < (it.i + 1) * DIRECT_FWD_ROWS ? F.nb6 : (it.i + 1) * DIRECT_FWD_ROWS;
  const double* __restrict__ G = a.fact + F.fact_off + (int64_t)F.ns6 * F.ns6;
  // 4 rows at a time: their loads are in flight together
  for (int r = it.i * DIRECT_FWD_ROWS + 4 * wave; r < r_end; r += 4 * (TPB / 64)) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    const double* g[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = G + (int64_t)(r + k < r_end ? r + k : r_end - 1) * F.ns6;
    for (int c = 2 * lane; c < F.ns6; c += 128) {
      const double2 bv = *reinterpret_cast<const double2*>(b + c);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double2 gv = *reinterpret_cast<const double2*>(g[k] + c);
        s[k] += gv.x * bv.x + gv.y * bv.y;
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o, 64);
    if (lane < 4 && r + lane < r_end) {
      const int row = r + lane, q = row / 6;
      const double dot = lane == 0 ? s[0] : lane == 1 ? s[1] : lane == 2 ? s[2] : s[3];
      a.v[F.v_off + row] = children(ns + q, row - 6 * q) - dot;
    }
  }
}

// Down: 32 columns of x_S = -(panel^T [b_S; x_B]), the panel's rows dealt to 16 groups of lanes.
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
  for (int base = 0; base < rows; base += BWD_CHUNK) {
    const int n = rows - base < BWD_CHUNK ? rows - base : BWD_CHUNK;
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += BWD_TPB) {
      const int r = base + k, q = r / 6;
      y[k] = r < F.ns6 ? a.b[F.b_off + r]
                       : a.sol[6 * (int64_t)a.nodes[F.nodes_off + q] + r - 6 * q];
    }
    __syncthreads();
    int k = g;
    for (; k + 7 * BWD_GROUPS < n; k += 8 * BWD_GROUPS) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = P[(int64_t)(base + k + u * BWD_GROUPS) * F.ns6];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u] * y[k + u * BWD_GROUPS];
    }
    for (; k < n; k += BWD_GROUPS) s += P[(int64_t)(base + k) * F.ns6] * y[k];
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

template <class Fn>
hipError_t launch_step(const DirectPlan& pl, int level, int step, Fn launch) {
  const DirectRange r = pl.steps[pl.level_off[level] + step];
  if (r.cnt == 0) return hipSuccess;
  launch(dim3((unsigned)r.cnt), r.off);
  return hipGetLastError();
}

}  // namespace

#define SSO_TRY(x)                 \
  do {                             \
    hipError_t e_ = (x);           \
    if (e_ != hipSuccess) return e_; \
  } while (0)

hipError_t launch_direct_factor(const DirectPlan& pl, const DirectArgs& a, hipStream_t s) {
  const DirectArgs* none = nullptr;
  for (int h = 0; h < pl.levels(); ++h) {
    SSO_TRY(launch_step(pl, h, STEP_ASM, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_assemble, g, dim3(TPB), 0, s, a, none, off, h);
    }));
    for (int p = 0; p < pl.level_np[h]; ++p) {
      SSO_TRY(launch_step(pl, h, STEP_PANEL + 2 * p, [&](dim3 g, int off) {
        hipLaunchKernelGGL(k_front_scale, g, dim3(TPB), 0, s, a, none, off, h, p);
      }));
      SSO_TRY(launch_step(pl, h, STEP_PANEL + 2 * p + 1, [&](dim3 g, int off) {
        hipLaunchKernelGGL(k_front_update, g, dim3(TPB), 0, s, a, none, off, h, p);
      }));
    }
    SSO_TRY(launch_step(pl, h, STEP_SCHUR, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_schur, g, dim3(TPB), 0, s, a, none, off, h);
    }));
  }
  return hipSuccess;
}

hipError_t launch_direct_solve(const DirectPlan& pl, const DirectArgs& a, hipStream_t s) {
  const DirectArgs* none = nullptr;
  for (int h = 0; h < pl.levels(); ++h)
    SSO_TRY(launch_step(pl, h, STEP_FWD, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_forward, g, dim3(TPB), 0, s, a, none, off, h);
    }));
  for (int h = pl.levels() - 1; h >= 0; --h)
    SSO_TRY(launch_step(pl, h, STEP_BWD, [&](dim3 g, int off) {
      hipLaunchKernelGGL(k_front_backward, g, dim3(BWD_TPB), 0, s, a, none, off, h);
    }));
  return hipSuccess;
}

}  // namespace sso
