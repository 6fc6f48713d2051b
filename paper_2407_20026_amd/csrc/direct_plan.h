// Plan of the sparse direct solver: nested dissection of the node graph and the fronts of a
// multifrontal elimination, with the work lists of its kernels.  Host code; built once per
// topology from the block pattern of K alone (never from coordinates, so that every problem of a
// topology eliminates in the same order and gives the same bits).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <vector>

namespace sso {

// Panel width of the elimination inside a front, and the rows of a work item of its kernels.
constexpr int DIRECT_NB = 64;
// Columns of a backward-substitution work item; rows of a forward-substitution one: one pass of a
// workgroup, or more, up to DIRECT_FWD_MOST, where the level has more than DIRECT_FWD_ITEMS passes
// for each (an item gathers the front's right-hand side for itself).
constexpr int DIRECT_BWD_COLS = 32;
constexpr int DIRECT_FWD_ROWS = 16;
constexpr int DIRECT_FWD_ITEMS = 2048;
constexpr int DIRECT_FWD_MOST = 4;
// Most own DOFs of a front (a substitution stages them in LDS).
constexpr int DIRECT_MAX_OWN = 6144;
// Most boundary DOFs of a front (byte offsets within its Schur complement have 32 bits).
constexpr int DIRECT_MAX_BOUNDARY = 32766;

// One front: ns own nodes (eliminated here), nb boundary nodes (ancestors' nodes that the front's
// subtree touches).  Its rows are the DOFs of the own nodes, then of the boundary nodes; its
// columns those of the own nodes.  Offsets are in values of the array named.
struct DirectFront {
  int32_t ns6, nb6;          // 6 ns, 6 nb
  int32_t nodes_off;         // own nodes, then boundary nodes (global node numbers)
  int32_t map_off;           // for each of its ns + nb nodes: position in child 0's boundary or
                             //   -1; then the same for child 1
  int32_t child[2];          // fronts, -1: none
  int32_t np;                // panels: ceil(ns6 / DIRECT_NB)
  int32_t nt;                // row tiles: np, then ceil(nb6 / DIRECT_NB)
  int32_t level;             // height: every child has a lower level
  int32_t tile_off;          // its row tiles' ends in tile_end
  int32_t e0, e1;            // entries of its first tile
  int32_t gain;              // its boundary rows are formed by the level's gain step
  int32_t pad;
  int64_t fact_off;          // factor [(ns6 + nb6) x ns6]
  int64_t work_off;          // assembled columns of the level, same shape
  int64_t again_off;         // np > 1: second work panel of the level, same shape
  int64_t w_off;             // np > 1: scaled panels of two steps, DIRECT_NB x DIRECT_NB row tiles,
                             //   and the last one's boundary tiles before they are scaled
  int64_t child_u[2];        // the children's u_off, 0 without a child
  int64_t u_off;             // Schur complement, lower triangle row by row (direct_tri)
  int64_t v_off;             // update vector of the forward substitution [nb6]
  int64_t b_off;             // right-hand side of the own DOFs [ns6]
};

// Entries of a lower triangle in front of row r, and of the triangle of r rows.
#ifdef __HIPCC__
__host__ __device__
#endif
inline int64_t direct_tri(int r) { return (int64_t)r * (r + 1) / 2; }

// Rows of row tile i of a front: own rows first, boundary rows in tiles of their own.
struct DirectRows {
  int32_t r0, n;
};
#ifdef __HIPCC__
__host__ __device__
#endif
inline DirectRows direct_rows(const DirectFront& F, int i) {
  DirectRows t;
  if (i < F.np) {
    t.r0 = i * DIRECT_NB;
    t.n = F.ns6 - t.r0;
  } else {
    t.r0 = F.ns6 + (i - F.np) * DIRECT_NB;
    t.n = F.ns6 + F.nb6 - t.r0;
  }
  if (t.n > DIRECT_NB) t.n = DIRECT_NB;
  return t;
}

// A work item: the front and up to two tile indices; K's entries [e0, e1) of tile (i, max(j, 0))
// in the first panel step; boundary rows [i, e0) in the forward substitution; e0 = 1 in the Schur
// step: tile (i, j) is updated with the last panel instead.
struct DirectItem {
  int32_t front, i, j, e0, e1;
};

// One 6x6 block of K in a tile of a front (a block across tiles is listed in each): where its first
// row and column lie in the tile, plus DIRECT_EDGE each, and its value slot (the block of (column
// node, row node), read transposed: K is bitwise symmetric).
constexpr int DIRECT_EDGE = 8;
struct DirectEntry {
  int32_t rc;                // row << 16 | column
  int32_t slot;
};

struct DirectRange {
  int32_t off, cnt;
};

// Workgroups go to the chip's XCDs, each with an L2 of its own, in turn.
constexpr int DIRECT_XCDS = 8;

// Step lists of a level: Schur complement, forward and backward substitution, then the panel steps
// 0 .. np: step q scales panel q (items with j < 0: row tile i) and updates with panel q - 1 (tile
// i, j).  Step 0 assembles as well, tiles on the diagonal and below it (those above it are their
// transposes): its items with j < 0 the first column of tiles, -j row tiles from i on; the others
// tile (i, j).  The update with the last panel goes with the Schur step, which does not wait for
// it.  On a level with a gain step, which does, it is panel step np, and
// the panel steps take the own rows only, the first one's boundary tiles being assembled like the
// others, and the gain step forms the boundary rows G.
enum { STEP_SCHUR = 0, STEP_FWD = 1, STEP_BWD = 2, STEP_GAIN = 3, STEP_PANEL = 4 };
// Boundary tiles that a panel step would update, from which on a level with several panels takes the
// gain step: four for each of the 256 CUs.  A level with 1740 (four fronts, 900 own DOFs) took 15 x
// 60 us without it and 15 x 28 + 286 with it; one with 870 (two fronts) 15 x 32 and 15 x 25 + 178.
constexpr int DIRECT_GAIN_TILES = 1024;
// Row tiles of a scaling item of step 0: one, so that a front's tiles spread over the chip, or as
// many, up to DIRECT_FIRST_MOST, as leave the level no more items than the chip holds at a time (each
// inverts the pivot block for itself, 17 us before its first tile and 5 for each one more).
constexpr int DIRECT_FIRST_ITEMS = 512;
constexpr int DIRECT_FIRST_MOST = 8;

struct DirectPlan {
  std::vector<DirectFront> fronts;    // level by level, leaves first
  std::vector<int32_t> nodes, maps;
  std::vector<DirectEntry> entries;
  std::vector<int32_t> tile_end;      // per row tile: end of the entries of its first tile
  std::vector<DirectItem> items;
  std::vector<DirectRange> steps;     // steps[level_off[h] + STEP_*] (panels: STEP_PANEL + q)
  std::vector<int32_t> level_off;     // per level
  std::vector<int32_t> level_np;      // most panels of a front of the level
  std::vector<int32_t> level_own;     // most own DOFs
  int n_nodes = 0;
  int64_t fact_len = 0, work_len = 0, again_len = 0, w_len = 0, u_len = 0, v_len = 0;
  // values of a problem's numeric arrays: the five above, v, and two vectors of all DOFs
  int64_t values() const {
    return fact_len + work_len + again_len + w_len + u_len + v_len + 12 * (int64_t)n_nodes;
  }
  int levels() const { return (int)level_off.size(); }
};

// Builds the plan for a block pattern (brow_ptr [n + 1], bcol, columns of a row ascending, the
// pattern symmetric).  Returns false when its numeric arrays would take more than max_bytes or a
// front has more than DIRECT_MAX_OWN own or DIRECT_MAX_BOUNDARY boundary DOFs, and soon after *stop
// (if given) is set.
bool build_direct_plan(int n, const int32_t* brow_ptr, const int32_t* bcol, double max_bytes,
                       DirectPlan& plan, const std::atomic<bool>* stop = nullptr);
// 0 when every invariant of the plan holds, else the number of the first failed check, with a
// message in msg.
int check_direct_plan(int n, const int32_t* brow_ptr, const int32_t* bcol,
                      const DirectPlan& plan, char* msg, size_t len);

}  // namespace sso
