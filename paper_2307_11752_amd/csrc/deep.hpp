// deep.hpp -- host side of the many-steps-per-pass kernel for D2Q9.  Internal.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "lattice.hpp"

// Split of a lattice into regions of RX x RY cells (RX = 2^log_rx), one per
// work-group; a pass of k steps completes the cells that
// lie k - 1 or more from a region's edge.
struct DeepPlan {
  bool use = false;
  int log_rx = 0, RY = 0;
  int steps = 0;  // steps of a pass at most
  double cost = 1e300;  // estimated us of a step
};

struct DeepLaunch {
  const DeepPlan* plan;
  int nx, ny;
  lbm::PopIndex pix;
  int steps;  // of this pass
  const void* src;
  void* dst;
  const uint32_t* link;
  const uint32_t* mov;
  int entry;  // src in natural form
  int exit;   // dst in natural form
  hipStream_t stream;
};

namespace lbm_detail {
DeepPlan make_deep_plan(int nx, int ny, size_t s, int num_cu);

// Cells that each region completes in a pass of `steps` steps, regions in a row
// of them and in all.
void deep_regions(const DeepPlan& plan, int nx, int ny, int steps, int* cx, int* cy, int* ntx,
                  int* nblocks);

template <typename S>
void launch_deep(bool shifted, bool masked, const DeepLaunch& a,
                 const lbm::StepParams<typename lbm::Store<S>::T>& p);
}  // namespace lbm_detail
