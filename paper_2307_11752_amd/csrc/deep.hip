// deep.hip -- many time steps of a D2Q9 lattice in one pass over the populations.
//
// A two-dimensional lattice is small: a step of it takes less time than the
// launch and the first access of a kernel do.  So a work-group takes a region of the
// lattice, keeps the populations of its cells in registers and advances them k
// steps, passing the moving ones on through LDS; the cells whose inputs would
// come from outside the region drop out, one ring a step, and the rest, k - 1 or
// more from the edge, is written.  Regions overlap by 2 (k - 1) cells.
//
// A thread holds C cells, a column of the region NT / RX rows apart.  LDS holds
// the eight moving post-collision populations of the region, twice where that
// fits (one barrier a step, else two).  Intermediate values are rounded to the
// storage type as a stored step would round them.  src and dst must differ: a
// work-group reads cells that its neighbours write.
#include <hip/hip_runtime.h>

#include "deep.hpp"
#include "handle.hpp"
#include "lattice.hpp"
#include "lbm.h"

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

constexpr int Q = 9;

template <int BYTES>
struct Raw;
template <>
struct Raw<2> { using U = uint16_t; };
template <>
struct Raw<4> { using U = uint32_t; };
template <>
struct Raw<8> { using U = uint64_t; };

struct DeepGeom {
  int nx, ny, log_rx, RY, steps;
  int narrow;  // the region exceeds the lattice on an axis
  int CX, CY, ntx, nblocks;  // cells a region completes, regions per row of them and in all
  PopIndex pix;
};

// EXIT: dst is left in natural form (as in pair_path.hpp).  A template parameter: as a
// run-time flag it cost every pass registers (1979 x 711 FP32, 47 steps: 517.6
// against 509.0 us).
template <typename S, bool SHIFT, bool MASKED, int NT, int C, bool EXIT>
__global__ void __launch_bounds__(NT)
    deep_kernel(const S* __restrict__ src, S* __restrict__ dst, const uint32_t* __restrict__ link,
                const uint32_t* __restrict__ mov, DeepGeom G, int entry,
                StepParams<typename Store<S>::T> p) {
  using T = typename Store<S>::T;
  using U = typename Raw<(int)sizeof(S)>::U;
  using V = Vel<Q>;
  constexpr int REGION = NT * C;
  constexpr int PAD = 66;  // rows of up to 64 cells: neighbours of cells at the edge stay in bounds
  constexpr bool TWICE = 2 * (Q - 1) * (REGION + 2 * PAD) * sizeof(U) <= 163840;
  __shared__ U tile[TWICE ? 2 : 1][Q - 1][REGION + 2 * PAD];

  const int per = (G.nblocks + 7) >> 3;  // neighbouring regions on one XCD
  const int id = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  if (id >= G.nblocks) return;  // the grid is a multiple of 8
  const int ty = id / G.ntx, tx = id - ty * G.ntx;
  const int RX = 1 << G.log_rx, k1 = G.steps - 1;
  const int lx = (int)threadIdx.x & (RX - 1), ly0 = (int)threadIdx.x >> G.log_rx;
  const int rows = NT >> G.log_rx;  // between a thread's cells
  const auto wrap = [&](int v, int n) {
    if (G.narrow) v %= n;  // the region is wider than the lattice
    return v < 0 ? v + n : (v >= n ? v - n : v);
  };
  const int x = wrap(tx * G.CX - k1 + lx, G.nx);
  const int xm = x == 0 ? G.nx - 1 : x - 1, xp = x == G.nx - 1 ? 0 : x + 1;
  // What a wall reflects waits in slot i of the cell itself.  Small regions are
  // bound by latency and load it beside the neighbour's population, before the
  // link word is known.
  constexpr bool BOTH = MASKED && C <= 2;
  T f[C][Q];
  uint32_t lw[C], mv[C];
  uint32_t own[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int y = wrap(ty * G.CY - k1 + ly0 + c * rows, G.ny);
    const int ym = y == 0 ? G.ny - 1 : y - 1, yp = y == G.ny - 1 ? 0 : y + 1;
    const uint32_t cell = (uint32_t)G.nx * (uint32_t)y + (uint32_t)x;
    own[c] = cell;
    lw[c] = MASKED ? link[cell] : 0u;
    mv[c] = MASKED && p.has_moving ? mov[cell] : 0u;
    const int X[3] = {entry ? x : xp, x, entry ? x : xm};  // x - c_i by c_i + 1
    const uint32_t Y[3] = {(uint32_t)G.nx * (uint32_t)(entry ? y : yp), (uint32_t)G.nx * (uint32_t)y,
                           (uint32_t)G.nx * (uint32_t)(entry ? y : ym)};
    T reflected[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const uint32_t from = G.pix.at(entry ? i : V::opp[i], Y[V::cy[i] + 1] + (uint32_t)X[V::cx[i] + 1]);
      const bool wall = MASKED && i > 0 && ((lw[c] >> (V::opp[i] - 1)) & 1u);
      f[c][i] = Store<S>::load(src + (BOTH || !wall ? from : G.pix.at(i, cell)));
      if (BOTH && i > 0) reflected[i] = Store<S>::load(src + G.pix.at(i, cell));
    }
#pragma unroll
    for (int i = 1; i < Q; ++i)
      if (BOTH) f[c][i] = (lw[c] >> (V::opp[i] - 1)) & 1u ? reflected[i] : f[c][i];
    if (MASKED && !(lw[c] & LINK_HAS_MOVING)) mv[c] = 0u;
  }
  const auto as_u = [](T t) {
    const S v = Store<S>::pack(t);
    U u;
    __builtin_memcpy(&u, &v, sizeof(S));
    return u;
  };
  const auto as_t = [](U u) {
    S v;
    __builtin_memcpy(&v, &u, sizeof(S));
    return Store<S>::cvt(v);
  };
  // Rows that dropped out are skipped in lattices with walls where a thread has
  // several (1024 x 512 FP32 4.6 against 5.4 us a step; a 2048 x 1024 box 12.1
  // against 11.7 without); what the cells outside compute else is read by cells
  // outside only.
  constexpr bool DROP = MASKED && C > 1;
  const int at0 = PAD + (int)threadIdx.x;
  for (int s = 0;; ++s) {
    const int buf = TWICE ? s & 1 : 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int ly = ly0 + c * rows;
      if (DROP && (ly < s || ly >= G.RY - s)) continue;
      const T rho = collide<Q, SHIFT, T>(f[c], p, MASKED && ((p.fused_u >> (s & 1)) & 1));
      if (MASKED && p.has_moving) {
#pragma unroll
        for (int i = 1; i < Q; ++i)
          if ((mv[c] >> (i - 1)) & 1u) f[c][i] = reflect_moving(f[c][i], rho, p.mw[i]);
      }
      if (s < k1) {
        f[c][0] = as_t(as_u(f[c][0]));
#pragma unroll
        for (int i = 1; i < Q; ++i) {
          const U u = as_u(f[c][i]);
          f[c][i] = as_t(u);
          tile[buf][i - 1][at0 + c * NT] = u;
        }
      }
    }
    if (s == k1) break;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int ly = ly0 + c * rows;
      if (DROP && (ly <= s || ly >= G.RY - s - 1)) continue;
      T g[Q];
#pragma unroll
      for (int i = 1; i < Q; ++i) {
        const T v = as_t(tile[buf][i - 1][at0 + c * NT - V::cx[i] - V::cy[i] * RX]);
        g[i] = MASKED && ((lw[c] >> (V::opp[i] - 1)) & 1u) ? f[c][V::opp[i]] : v;
      }
#pragma unroll
      for (int i = 1; i < Q; ++i) f[c][i] = g[i];
    }
    if (!TWICE) __syncthreads();
  }
  if (lx < k1 || lx >= k1 + G.CX || tx * G.CX + lx - k1 >= G.nx) return;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int ly = ly0 + c * rows;
    if (ly < k1 || ly >= k1 + G.CY || ty * G.CY + ly - k1 >= G.ny) continue;
    if (!EXIT) {
#pragma unroll
      for (int i = 0; i < Q; ++i) Store<S>::store(dst + G.pix.at(V::opp[i], own[c]), f[c][i]);
      continue;
    }
    // natural form: into slot i of x + c_i, or, reflected by a wall, slot opp(i) of x
    if (MASKED && !(lw[c] & LINK_FLUID)) continue;
    const int y = ty * G.CY + ly - k1;
    const int X[3] = {xm, x, xp};  // x + c_i by c_i + 1
    const uint32_t Y[3] = {(uint32_t)G.nx * (uint32_t)(y == 0 ? G.ny - 1 : y - 1), (uint32_t)G.nx * (uint32_t)y,
                           (uint32_t)G.nx * (uint32_t)(y == G.ny - 1 ? 0 : y + 1)};
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const bool wall = MASKED && i > 0 && ((lw[c] >> (i - 1)) & 1u);
      const uint32_t away = G.pix.at(i, Y[V::cy[i] + 1] + (uint32_t)X[V::cx[i] + 1]);
      Store<S>::store(dst + (wall ? G.pix.at(V::opp[i], own[c]) : away), f[c][i]);
    }
  }
}

template <bool SHIFT, bool MASKED, int NT, int C, bool EXIT>
void launch(const DeepLaunch& a, const StepParams<typename Store<Stored>::T>& p) {
  const DeepPlan& P = *a.plan;
  DeepGeom G{};
  G.nx = a.nx;
  G.ny = a.ny;
  G.log_rx = P.log_rx;
  G.RY = P.RY;
  G.steps = a.steps;
  lbm_detail::deep_regions(P, a.nx, a.ny, a.steps, &G.CX, &G.CY, &G.ntx, &G.nblocks);
  G.narrow = (1 << P.log_rx) > a.nx || P.RY > a.ny;
  G.pix = a.pix;
  hipLaunchKernelGGL((deep_kernel<Stored, SHIFT, MASKED, NT, C, EXIT>), dim3((unsigned)((G.nblocks + 7) / 8 * 8)),
                     dim3(NT), 0, a.stream, (const Stored*)a.src, (Stored*)a.dst, a.link, a.mov, G,
                     a.entry, p);
}

template <bool SHIFT, bool MASKED, int NT, int C>
void launch(const DeepLaunch& a, const StepParams<typename Store<Stored>::T>& p) {
  a.exit ? launch<SHIFT, MASKED, NT, C, true>(a, p) : launch<SHIFT, MASKED, NT, C, false>(a, p);
}

template <bool SHIFT, bool MASKED>
void launch(const DeepLaunch& a, const StepParams<typename Store<Stored>::T>& p) {
  const int cells = a.plan->RY << a.plan->log_rx;
  if (cells == 256) return launch<SHIFT, MASKED, 256, 1>(a, p);
  if (cells == 512) return launch<SHIFT, MASKED, 512, 1>(a, p);
  if (cells == 1024) return launch<SHIFT, MASKED, 1024, 1>(a, p);
  if (cells == 2048 || sizeof(Stored) == 8) return launch<SHIFT, MASKED, 1024, 2>(a, p);
  launch<SHIFT, MASKED, 1024, sizeof(Stored) == 8 ? 2 : 4>(a, p);
}

}  // namespace

template <>
void lbm_detail::launch_deep<Stored>(bool shifted, bool masked, const DeepLaunch& a,
                                     const StepParams<typename Store<Stored>::T>& p) {
  if (shifted)
    masked ? launch<true, true>(a, p) : launch<true, false>(a, p);
  else
    masked ? launch<false, true>(a, p) : launch<false, false>(a, p);
}
