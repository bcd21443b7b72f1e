// deep_plan.hip -- regions of the many-steps-per-pass D2Q9 kernel (host only).
#include <algorithm>

#include "deep.hpp"

namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }

}  // namespace

void lbm_detail::deep_regions(const DeepPlan& P, int nx, int ny, int steps, int* CX, int* CY,
                              int* ntx, int* nblocks) {
  // as few regions as hold the lattice, of about the same size
  *CX = ceil_div(nx, ceil_div(nx, (1 << P.log_rx) - 2 * (steps - 1)));
  *CY = ceil_div(ny, ceil_div(ny, P.RY - 2 * (steps - 1)));
  *ntx = ceil_div(nx, *CX);
  *nblocks = *ntx * ceil_div(ny, *CY);
}

// The estimated time of a pass of k steps, in us: a launch, then for each
// round of work-groups loading and storing of the cells of a CU, and k steps of
// a fixed latency and a share by cells; and half the time of its bytes at 5 TB/s.  The constants are from timings of 40
// regions with 2 to 16 steps on nine lattices (64^2 to 2048 x 1024; FP64, FP32,
// BF16); the choice came out at most 9 % slower than the fastest region timed.
// Every lattice gains (us a step by single steps / two steps a pass over
// marching tiles / so): cavity 64^2 FP64 4.2 / 2.3 / 1.2, 730 x 150 FP32 4.5 /
// 3.2 / 1.8, 1024 x 512 FP32 - / 7.1 / 4.6, 2048 x 1024 FP32 - / 18.5 / 11.7 and
// FP64 - / 32.0 / 28.0.
DeepPlan lbm_detail::make_deep_plan(int nx, int ny, size_t s, int num_cu) {
  DeepPlan best;
  const double per_cell = s == 8 ? 1.0e-3 : 0.75e-3, io = s == 8 ? 1.35e-3 : 1.05e-3;
  for (int cells = 256; cells <= (s == 8 ? 2048 : 4096); cells *= 2) {
    // work-groups of a CU: LDS, but for 16-bit storage, which the registers bound
    const size_t lds = 16 * (cells + 132) * s;
    const int per_cu = std::max(1, std::min((int)(163840 / lds), 2048 / std::min(cells, 1024)));
    for (int lr = 4; lr <= 6; ++lr) {
      DeepPlan P;
      P.use = true;
      P.log_rx = lr;
      P.RY = cells >> lr;
      if (P.RY < 8 || P.RY > 64) continue;
      for (P.steps = 2; P.steps <= 16; ++P.steps) {
        if (std::min(1 << lr, P.RY) - 2 * (P.steps - 1) < 2) break;
        int CX, CY, ntx, blocks;
        deep_regions(P, nx, ny, P.steps, &CX, &CY, &ntx, &blocks);
        const double rounds = ceil_div(blocks, num_cu * per_cu);
        const double of_cu = (double)cells * std::min(per_cu, ceil_div(blocks, num_cu));
        const double mem = 0.5 * 9.0 * s * ((double)blocks * cells + (double)nx * ny) / 5e6;
        P.cost = (2.3 + rounds * (io * of_cu + P.steps * (0.45 + per_cell * of_cu)) + mem) / P.steps;
        if (P.cost < best.cost) best = P;
      }
    }
  }
  return best;
}
