// pair.hip -- launches of the two-steps-per-pass kernel (pair_path.hpp).
//
// Compiled once per storage type (LBM_PAIR_STORAGE = LBM_STORE_*): the
// instantiations are the larger part of the library's build time.
#include <hip/hip_runtime.h>

#include "handle.hpp"
#include "lattice.hpp"
#include "lbm.h"
#include "pair.hpp"
#include "pair_path.hpp"

using namespace lbm;

namespace {

#if LBM_PAIR_STORAGE == 0
using Stored = double;
#elif LBM_PAIR_STORAGE == 1
using Stored = float;
#elif LBM_PAIR_STORAGE == 2
using Stored = _Float16;
#else
using Stored = bf16s;
#endif

// Blocks are dealt to the 8 XCDs in turn: XCD k takes the k-th eighth of the
// tiles (plane after plane of them), so that neighbouring tiles, which read
// each other's columns, share one L2.  TGV 256^3 FP32: 487 us a pass against
// 518 us in plain order (fetched bytes 1.06x the populations).
template <int Q, typename S, bool SHIFT, bool MASKED, bool SEP, bool SMALL, bool EXIT>
__global__ void __launch_bounds__((pair_columns<Q, S, SMALL>()))
    pair_kernel(const S* __restrict__ src, S* __restrict__ dst, const uint32_t* __restrict__ link,
                const uint32_t* __restrict__ mov, PairGeom G, int entry,
                StepParams<typename Store<S>::T> p) {
  const int per = (G.nblocks + 7) >> 3;
  const int id = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (id >= G.nblocks) return;  // the grid is a multiple of 8
  const int zc = id / G.tiles;
  const int z0 = zc * G.ZC;
  pair_pass<Q, S, SHIFT, MASKED, SEP, SMALL, EXIT>(src, dst, link, mov, G, entry != 0,
                                                   id - zc * G.tiles, z0, min(z0 + G.ZC, G.nz), p);
}

#if LBM_PAIR_STORAGE <= 1
// The same pass over a batch: one work-group per item of the work list.  Members
// differ in the columns of a tile, so waves past an item's last column end at
// once (a barrier waits for the surviving waves only).
template <int Q, typename S, bool SHIFT, bool SMALL, bool EXIT>
__global__ void __launch_bounds__((pair_columns<Q, S, SMALL>()))
    pair_batch_kernel(const S* __restrict__ src, S* __restrict__ dst,
                      const PairItem* __restrict__ items, int entry) {
  const PairItem& it = items[blockIdx.x];
  if (it.z0 == it.z1) return;
  const PairGeom G = it.geom;
  if (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) * 64 >= G.W * G.H) return;
  StepParams<typename Store<S>::T> p{};
  p.base = (typename Store<S>::T)Store<S>::unit;
  p.omega = (typename Store<S>::T)it.omega;
  pair_pass<Q, S, SHIFT, false, false, SMALL, EXIT>(src + it.pop_off, dst + it.pop_off, nullptr, nullptr,
                                                    G, entry != 0, it.tile, it.z0, it.z1, p);
}

template <int Q, bool SHIFT, bool EXIT>
void launch_batch(const PairBatchLaunch& a) {
  const auto kernel = a.small ? pair_batch_kernel<Q, Stored, SHIFT, true, EXIT>
                              : pair_batch_kernel<Q, Stored, SHIFT, false, EXIT>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)a.nitems), dim3((unsigned)a.threads), 0, a.stream,
                     (const Stored*)a.src, (Stored*)a.dst, a.items, a.entry);
}

template <int Q, bool SHIFT>
void launch_batch(const PairBatchLaunch& a) {
  a.exit ? launch_batch<Q, SHIFT, true>(a) : launch_batch<Q, SHIFT, false>(a);
}
#endif

template <bool SHIFT, bool MASKED, bool EXIT>
void launch(const PairLaunch& a, const StepParams<typename Store<Stored>::T>& p) {
  const PairGeom& G = a.plan->geom;
  const dim3 grid((unsigned)((G.nblocks + 7) / 8 * 8)), block((unsigned)((G.W * G.H + 63) / 64 * 64));
  const Stored* src = (const Stored*)a.src;
  Stored* dst = (Stored*)a.dst;
  const auto kernel = a.plan->small ? pair_kernel<19, Stored, SHIFT, MASKED, false, true, EXIT>
                      : MASKED && a.plan->separable
                          ? pair_kernel<19, Stored, SHIFT, MASKED, MASKED, false, EXIT>
                          : pair_kernel<19, Stored, SHIFT, MASKED, false, false, EXIT>;
  hipLaunchKernelGGL(kernel, grid, block, 0, a.stream, src, dst, a.link, a.mov, G, a.entry, p);
}

template <bool SHIFT, bool MASKED>
void launch(const PairLaunch& a, const StepParams<typename Store<Stored>::T>& p) {
  a.exit ? launch<SHIFT, MASKED, true>(a, p) : launch<SHIFT, MASKED, false>(a, p);
}

}  // namespace

template <>
void lbm_detail::launch_pair<Stored>(bool shifted, bool masked, const PairLaunch& a,
                                     const StepParams<typename Store<Stored>::T>& p) {
  if (shifted)
    masked ? launch<true, true>(a, p) : launch<true, false>(a, p);
  else
    masked ? launch<false, true>(a, p) : launch<false, false>(a, p);
}

#if LBM_PAIR_STORAGE <= 1
template <>
void lbm_detail::launch_pair_batch<Stored>(int q, bool shifted, const PairBatchLaunch& a) {
  if (q == 9)
    shifted ? launch_batch<9, true>(a) : launch_batch<9, false>(a);
  else
    shifted ? launch_batch<19, true>(a) : launch_batch<19, false>(a);
}
#endif
