// pair.hpp -- host side of the two-steps-per-pass kernel: its geometry and the
// choice of tiles.  Internal.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <vector>

#include "lattice.hpp"

// Geometry of one pass (march axis last: D2Q9 has ny = 1 and nz its rows).
// Byte offset of population i of cell r of plane z (r = x + nx y):
//   separable placements (whole planes per chunk, or one array per population):
//     i pb + z zb + s r + ((s r) >> sh) kb;
//   else, with c = s (r + z nx ny):  i pb + c + (c >> sh) kb  (PopIndex in bytes).
// (px instead of nx where rows are padded).
struct PairGeom {
  int nx, ny, nz;
  int px;               // cells from one stored row to the next
  int TX, TY, W, H;     // columns of a tile without and with its halo
  int ntx, tiles, ZC;   // tiles per row of tiles and per plane, planes per block
  int nblocks;
  uint32_t bytes;       // size of a population buffer
  uint32_t pb, zb, kb;
  int sh;
};

struct PairPlan {
  bool use = false;        // runs of steps take this path
  bool small = false;      // the kernel with the smaller column limit
  bool separable = false;
  double cost = 1e300;     // estimated us of a pass
  PairGeom geom{};
};

struct PairLaunch {
  const PairPlan* plan;
  const void* src;
  void* dst;
  const uint32_t* link;
  const uint32_t* mov;
  int entry;  // src in natural form
  int exit;   // dst in natural form
  hipStream_t stream;
};

// One work-group of a batch's pass: planes z0 .. z1 - 1 of a tile of a member
// (z0 == z1: nothing).
struct PairItem {
  PairGeom geom;
  int tile, z0, z1;
  uint64_t pop_off;  // elements from the start of the batch's populations
  double omega;
};

struct PairBatchLaunch {
  const PairItem* items;
  int nitems, threads;
  bool small;
  const void* src;
  void* dst;
  int entry, exit;
  hipStream_t stream;
};

// What the plan of a batch needs to know of a member.
struct PairMember {
  int nx, ny, nz, px;
  lbm::PopIndex pix;
  uint64_t pop_off;
  double omega;
};

// The work list of a batch's pass, in launch order; empty: it does not pay or apply.
struct PairBatchPlan {
  std::vector<PairItem> items;
  bool small = false;
  int threads = 0;
};

// Columns (threads) of a work-group at most: two planes of populations fit one
// CU's LDS (160 KB), or, small, several work-groups to a CU.
constexpr int pair_column_limit(int q, size_t s, bool small) {
  return q == 9 ? (small ? 64 : 256) : (s == 8 ? (small ? 192 : 512) : (small ? 320 : 704));
}

namespace lbm_detail {
// Tiles for a D3Q19 lattice of nx x ny x nz cells (host only; num_cu compute units).
// plan.use is false where the pass does not apply (a population buffer of
// 2^32 bytes or more) or does not pay.
PairPlan make_pair_plan(int nx, int ny, int nz, size_t s, bool masked,
                        const lbm::PopIndex& L, int num_cu);

PairBatchPlan make_pair_batch_plan(int q, size_t s, const std::vector<PairMember>& members,
                                   int num_cu);

template <typename S>
void launch_pair_batch(int q, bool shifted, const PairBatchLaunch& a);

template <typename S>
void launch_pair(bool shifted, bool masked, const PairLaunch& a,
                 const lbm::StepParams<typename lbm::Store<S>::T>& p);
}  // namespace lbm_detail
