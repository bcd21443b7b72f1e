// pair_path.hpp -- two time steps in one pass over the populations.
//
// Between two launches the populations lie in the swapped form of the AA
// pattern (slot opp(i) of x holds the post-collision g_i(x)), so a step is
// "gather g_i(x - c_i), collide, write g*(x) in place".  Two such steps need
// the first one's results at the neighbours of a cell only, so a work-group
// keeps them in LDS and the populations cross HBM once per two steps:
//
//   a work-group owns a tile of TX x TY columns and marches through ZC planes.
//   Interval z: every thread takes one column of the tile with a one-cell halo
//   (W x H = (TX + 2) x (TY + 2) columns), gathers the populations of plane z
//   from `src`, collides (step 1) and leaves the result in LDS; the threads of
//   the tile proper take plane z - 1 from LDS (neighbouring columns), which
//   completes the input of plane z - 2, collide (step 2) and write it to `dst`.
//
// LDS holds two planes, so one barrier per interval separates the planes
// written from the planes read; populations that move along the march wait in
// registers.  Step 2 is dealt to threads of its own (0 .. TX TY - 1), so that
// only whole waves idle in it.  Intermediate values are rounded to the storage
// type as a stored step would round them.
//
// The halo columns are collided by two or more work-groups; their populations
// come from L2 when neighbouring tiles run on one XCD, hence the block order.
// src and dst must differ: a work-group reads columns its neighbours write.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fluid_path.hpp"
#include "lattice.hpp"
#include "pair.hpp"

namespace lbm {

// Velocity components as the pass sees them: (px, py) in the tile's plane, m along the
// march.  D3Q19 marches along z with (x, y) tiles; D2Q9 along y with runs of x.
template <int Q>
struct March {
  using V = Vel<Q>;
  static constexpr int px(int i) { return V::cx[i]; }
  static constexpr int py(int i) { return V::D == 3 ? V::cy[i] : 0; }
  static constexpr int m(int i) { return V::D == 3 ? V::cz[i] : V::cy[i]; }
  static constexpr int count(int mm) {
    int n = 0;
    for (int i = 0; i < Q; ++i) n += m(i) == mm;
    return n;
  }
  static constexpr int rank(int i) {  // among the velocities of the same march component
    int n = 0;
    for (int k = 0; k < i; ++k) n += m(k) == m(i);
    return n;
  }
};

// A stored value: U as it lies in LDS, R in registers (16-bit values extended to
// a full register, or the compiler packs the ones that live across the loop in
// pairs, waiting for loads that are still on their way).
template <int BYTES>
struct BufValue;
template <>
struct BufValue<2> {
  using U = uint16_t;
  using R = uint32_t;
  static __device__ __forceinline__ R load(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    return __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0);
  }
  static __device__ __forceinline__ void store_nt(R x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b16((U)x, r, v, s, 2);
  }
  static __device__ __forceinline__ void store(R x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b16((U)x, r, v, s, 0);
  }
};
template <>
struct BufValue<4> {
  using U = uint32_t;
  using R = U;
  static __device__ __forceinline__ U load(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0);
  }
  static __device__ __forceinline__ void store_nt(U x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b32(x, r, v, s, 2);
  }
  static __device__ __forceinline__ void store(U x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b32(x, r, v, s, 0);
  }
};
template <>
struct BufValue<8> {
  using U = raw8;
  using R = U;
  static __device__ __forceinline__ U load(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    return __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0);
  }
  static __device__ __forceinline__ void store_nt(U x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b64(x, r, v, s, 2);
  }
  static __device__ __forceinline__ void store(U x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
    __builtin_amdgcn_raw_buffer_store_b64(x, r, v, s, 0);
  }
};

template <int Q, typename S, bool SMALL>
constexpr int pair_columns() {
  return pair_column_limit(Q, sizeof(S), SMALL);
}

template <typename V>
__device__ __forceinline__ void in_register(V& v) {
  asm volatile("" : "+v"(v));
}

// One pass of a work-group: tile `tl` of the plane, planes z0 .. z1 - 1.
//   entry: src is in natural form (slot i of x holds f_i(x)): step 1 takes its
//   own cell's slots (only scalar address parts depend on it).
//   EXIT: dst is left in natural form: step 2 writes what it sends to x + c_i into
//   slot i there, or, where a wall reflects it, into slot opp(i) of x; cells that
//   are not fluid send nothing.  Every slot of a fluid cell has one writer.  The
//   lines it writes are shared and written in part: 20 steps that end so, with a
//   field read, take 1 % longer (256^3 FP32 5386 against 5330 us) and 3 % (512 x
//   128 x 128 FP32 with walls 3096 against 3014).
//   SEP: separable placement.
template <int Q, typename S, bool SHIFT, bool MASKED, bool SEP, bool SMALL, bool EXIT>
__device__ __forceinline__ void pair_pass(const S* __restrict__ src, S* __restrict__ dst,
                                          const uint32_t* __restrict__ link,
                                          const uint32_t* __restrict__ mov, const PairGeom& G,
                                          bool entry, int tl, int z0, int z1,
                                          const StepParams<typename Store<S>::T>& p) {
  using T = typename Store<S>::T;
  using V = Vel<Q>;
  using M = March<Q>;
  using B = BufValue<(int)sizeof(S)>;
  using U = typename B::U;
  using R = typename B::R;
  constexpr int NC = pair_columns<Q, S, SMALL>();
  constexpr bool D3 = V::D == 3;
  constexpr uint32_t SB = (uint32_t)sizeof(S);
  __shared__ U tile[2][Q][NC];
  __shared__ uint32_t words[MASKED ? 2 : 1][MASKED ? NC : 1];

  const int tyi = tl / G.ntx, txi = tl - tyi * G.ntx;
  const int tid = (int)threadIdx.x;
  const auto dec = [](int v, int n) { return v == 0 ? n - 1 : v - 1; };
  const auto inc = [](int v, int n) { return v == n - 1 ? 0 : v + 1; };
  // planes -1 .. nz + 3 (there are at least four)
  const auto wrap = [&](int z) { return z < 0 ? z + G.nz : (z >= G.nz ? z - G.nz : z); };

  // Step 1: the column of this thread.  Threads past the last column and
  // columns past the far edge's halo repeat another column (same values).
  const int col = min(tid, G.W * G.H - 1);
  uint32_t nb[3][D3 ? 3 : 1];  // in-plane byte offsets (SEP) or s r of the neighbour columns
  uint32_t r1;
  {
    const int ly = D3 ? col / G.W : 0, lx = col - ly * G.W;
    int x = min(txi * G.TX + lx - 1, G.nx), y = D3 ? min(tyi * G.TY + ly - 1, G.ny) : 0;
    x = x < 0 ? G.nx - 1 : (x >= G.nx ? x - G.nx : x);
    if (D3) y = y < 0 ? G.ny - 1 : (y >= G.ny ? y - G.ny : y);
    const int X[3] = {entry ? x : dec(x, G.nx), x, entry ? x : inc(x, G.nx)};
    const int Y[3] = {entry || !D3 ? y : dec(y, G.ny), y, entry || !D3 ? y : inc(y, G.ny)};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < (D3 ? 3 : 1); ++b) {
        const uint32_t c = SB * ((uint32_t)G.px * (uint32_t)Y[D3 ? b : 1] + (uint32_t)X[a]);
        nb[a][b] = SEP ? c + __umul24(c >> G.sh, G.kb) : c;
      }
    r1 = (uint32_t)G.px * (uint32_t)y + (uint32_t)x;
  }
  constexpr int MID = D3 ? 1 : 0;
  const uint32_t np = (uint32_t)G.px * (uint32_t)G.ny;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, G.bytes, 0x00027000);
  // lane and scalar part of the address of in-plane offset o in plane z (slot 0)
  const auto lane_off = [&](uint32_t o, uint32_t z) {
    if (SEP) return o;
    const uint32_t c = o + z * (np * SB);
    return c + __umul24(c >> G.sh, G.kb);
  };
  const auto plane_off = [&](uint32_t z) { return SEP ? z * G.zb : 0u; };

  // Planes in flight: first(z) asks for plane z + AHEAD, two intervals ahead but
  // for FP64, whose two sets of registers would spill, and the last pass of a run
  // in natural form (512 x 128 x 128 FP32 with walls, 10 passes: 3105 us, 3165
  // with two; without walls the same).
  constexpr int AHEAD = sizeof(S) == 8 || EXIT ? 1 : 2;
  R sets[AHEAD][Q];
  R(&ra)[Q] = sets[0];
  R(&rb)[Q] = sets[AHEAD - 1];
  const auto load_plane = [&](R(&raw)[Q], int z, uint32_t lw) {
    z = wrap(z);
    const int Z[3] = {entry ? z : dec(z, G.nz), z, entry ? z : inc(z, G.nz)};
    if (MASKED && entry) lw = 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const uint32_t slot = (uint32_t)(entry ? i : V::opp[i]) * G.pb;
      const int zs = Z[1 - M::m(i)];
      const uint32_t o = nb[1 - M::px(i)][D3 ? 1 - M::py(i) : 0];
      if (!MASKED || i == 0) {
        raw[i] = B::load(rs, lane_off(o, zs), slot + plane_off(zs));
      } else {
        // a population reflected by a wall waits in slot i of the cell itself
        const uint32_t from = lane_off(o, zs) + (slot + plane_off(zs));
        const uint32_t own = lane_off(nb[1][MID], Z[1]) + ((uint32_t)i * G.pb + plane_off(Z[1]));
        raw[i] = B::load(rs, (lw >> (V::opp[i] - 1)) & 1u ? own : from, 0);
      }
    }
  };
  // link words of this thread's column in planes z, z + 1 and z + 2 before first(z);
  // the last may still be on its way
  uint32_t w0 = 0, w1 = 0, w2 = 0;
  const __amdgpu_buffer_rsrc_t rl =
      __builtin_amdgcn_make_buffer_rsrc((void*)link, 0, MASKED ? np * (uint32_t)G.nz * 4u : 0u, 0x00027000);
  const auto load_link = [&](int z) -> uint32_t {
    if (!MASKED) return 0u;
    return __builtin_amdgcn_raw_buffer_load_b32(rl, r1 * 4u, (uint32_t)wrap(z) * (np * 4u), 0);
  };
  // post-collision correction of the populations a moving wall reflects
  const auto moving = [&](T(&f)[Q], T rho, uint32_t lw, uint32_t cell) {
    if (MASKED && p.has_moving) {
      const uint32_t mv = lw & LINK_HAS_MOVING ? mov[cell] : 0u;
#pragma unroll
      for (int i = 1; i < Q; ++i)
        if ((mv >> (i - 1)) & 1u) f[i] = reflect_moving(f[i], rho, p.mw[i]);
    }
  };
  const auto as_t = [](R r) {
    const U u = (U)r;
    S v;
    __builtin_memcpy(&v, &u, sizeof(S));
    return Store<S>::cvt(v);
  };
  const auto as_u = [](T t) {
    const S v = Store<S>::pack(t);
    U u;
    __builtin_memcpy(&u, &v, sizeof(S));
    return u;
  };
  const auto first = [&](R(&raw)[Q], int z, bool again) {  // step 1 of plane z into LDS
    T f[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) f[i] = as_t(raw[i]);
    const uint32_t w = w0;
    w0 = w1;
    w1 = w2;
    if (again) {
      w2 = load_link(z + 3);
      load_plane(raw, z + AHEAD, AHEAD == 2 ? w1 : w0);
    }
    __builtin_amdgcn_sched_barrier(0);
    const T rho = collide<Q, SHIFT, T>(f, p, MASKED && (p.fused_u & 1));
    if (MASKED) {
      moving(f, rho, w, r1 + np * (uint32_t)wrap(z));
      words[z & 1][col] = w;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) tile[z & 1][i][col] = as_u(f[i]);
  };

  w0 = load_link(z0 - 1);
  w1 = load_link(z0);
  w2 = load_link(z0 + 1);
  load_plane(ra, z0 - 1, w0);
  if (AHEAD == 2) load_plane(rb, z0, w1);
  const auto more = [&](int z) { return z + AHEAD <= z1; };

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (wave * 64 >= G.TX * G.TY) {  // no column in step 2
    int z = z0 - 1;
    for (; z + 3 <= z1; z += 2) {
      first(ra, z, true);
      __syncthreads();
      first(rb, z + 1, true);
      __syncthreads();
    }
    first(ra, z, more(z));  // two or three planes left
    __syncthreads();
    first(rb, z + 1, more(z + 1));
    __syncthreads();
    if (z + 2 <= z1) {
      first(ra, z + 2, false);
      __syncthreads();
    }
    return;
  }

  // Step 2: the column of this thread in the tile proper (threads past the
  // last one, and columns past the edge, repeat another)
  const int t2 = min(tid, G.TX * G.TY - 1);
  int cx2, cy2;
  {
    cy2 = D3 ? t2 / G.TX : 0;
    cx2 = t2 - cy2 * G.TX;
    cx2 = min(cx2, G.nx - 1 - txi * G.TX);
    if (D3) cy2 = min(cy2, G.ny - 1 - tyi * G.TY);
  }
  const uint32_t r2 = (uint32_t)G.px * (uint32_t)(D3 ? tyi * G.TY + cy2 : 0) + (uint32_t)(txi * G.TX + cx2);
  // in-plane byte offset of row-and-column r2 (as nb)
  const auto in_plane = [&](uint32_t r) {
    return SEP ? r * SB + __umul24((r * SB) >> G.sh, G.kb) : r * SB;
  };
  const uint32_t out0 = in_plane(r2);
  const int c2 = (D3 ? (cy2 + 1) * G.W : 0) + cx2 + 1;
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(dst, 0, G.bytes, 0x00027000);

  constexpr int N0 = M::count(0), N1 = M::count(1);
  // inputs of plane z - 2 / z - 1 that are known before plane z is: h0 / hA the
  // populations of plane z - 2 (resting and up-going), hB the up-going ones of
  // plane z - 1; hS: the up-going post-collision values of the cell itself at z - 2
  R h0[N0], hA[N1], hB[N1], hS[MASKED ? N1 : 1];
  uint32_t lwR = 0;
  const auto second = [&](int z, bool out) {
    const int buf = (z - 1) & 1;
    const uint32_t lwP = MASKED ? words[buf][c2] : 0u;
    const auto take = [&](int i) -> R {
      return tile[buf][i][c2 - M::px(i) - (D3 ? M::py(i) * G.W : 0)];
    };
    if (out) {
      T e[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        if (M::m(i) < 0) {
          R v = take(i);
          if (MASKED && ((lwR >> (V::opp[i] - 1)) & 1u)) v = hS[M::rank(V::opp[i])];
          e[i] = as_t(v);
        } else {
          e[i] = as_t(M::m(i) == 0 ? h0[M::rank(i)] : hA[M::rank(i)]);
        }
      }
      const T rho = collide<Q, SHIFT, T>(e, p, MASKED && (p.fused_u & 2));
      moving(e, rho, lwR, r2 + np * (uint32_t)(z - 2));
      const uint32_t vo = lane_off(out0, (uint32_t)(z - 2)), so = plane_off((uint32_t)(z - 2));
      if constexpr (EXIT) {
        // the neighbours' places are computed anew: held across the loop they
        // cost 9 registers that the walled kernels do not have
        int x = txi * G.TX + cx2, y = D3 ? tyi * G.TY + cy2 : 0;
        in_register(x);
        in_register(y);
        const int X[3] = {dec(x, G.nx), x, inc(x, G.nx)};
        const int Y[3] = {D3 ? dec(y, G.ny) : 0, y, D3 ? inc(y, G.ny) : 0};
        const int Z[3] = {dec(z - 2, G.nz), z - 2, inc(z - 2, G.nz)};
        if (!MASKED || (lwR & LINK_FLUID)) {
#pragma unroll
          for (int i = 0; i < Q; ++i) {
            const uint32_t zd = (uint32_t)Z[1 + M::m(i)];
            const uint32_t away = lane_off(
                in_plane((uint32_t)G.px * (uint32_t)Y[1 + M::py(i)] + (uint32_t)X[1 + M::px(i)]), zd);
            const uint32_t there = plane_off(zd) + (uint32_t)i * G.pb;
            uint32_t at = away, base = there;
            if (MASKED && i > 0) {
              at = (lwR >> (i - 1)) & 1u ? vo + (so + (uint32_t)V::opp[i] * G.pb) : away + there;
              base = 0;
            }
            // rows that are shifted along x share lines with the next tile's, which L2 joins
            M::px(i) ? B::store(as_u(e[i]), rd, at, base) : B::store_nt(as_u(e[i]), rd, at, base);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) B::store_nt(as_u(e[i]), rd, vo, (uint32_t)V::opp[i] * G.pb + so);
      }
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if (M::m(i) == 0) {
        if (MASKED && i > 0)
          h0[M::rank(i)] = (lwP >> (V::opp[i] - 1)) & 1u ? (R)tile[buf][V::opp[i]][c2] : take(i);
        else
          h0[M::rank(i)] = take(i);
      }
      if (M::m(i) > 0) {
        hA[M::rank(i)] = hB[M::rank(i)];
        if (MASKED) {
          if ((lwP >> (V::opp[i] - 1)) & 1u) hA[M::rank(i)] = tile[buf][V::opp[i]][c2];
          hS[M::rank(i)] = tile[buf][i][c2];
        }
        hB[M::rank(i)] = take(i);
      }
    }
    lwR = lwP;
    // the values are in registers before the barrier that lets others overwrite
    // their place (the compiler may otherwise move the reads past it)
#pragma unroll
    for (int k = 0; k < N0; ++k) in_register(h0[k]);
#pragma unroll
    for (int k = 0; k < N1; ++k) {
      in_register(hA[k]);
      in_register(hB[k]);
      if (MASKED) in_register(hS[k]);
    }
    in_register(lwR);
  };
  const auto both = [&](R(&raw)[Q], int z, bool again, bool out) {
    first(raw, z, again);
    __builtin_amdgcn_sched_barrier(0);
    second(z, out);
    __syncthreads();
  };
  // In the loop every load and store is unconditional, so that the count of
  // outstanding accesses is known and waiting for a plane waits for nothing
  // issued after it.
  first(ra, z0 - 1, true);
  __syncthreads();
  both(rb, z0, more(z0), false);
  both(ra, z0 + 1, more(z0 + 1), false);
  int z = z0 + 2;
  for (; z + 3 <= z1; z += 2) {
    both(rb, z, true, true);
    both(ra, z + 1, true, true);
  }
  if (z <= z1) both(rb, z, more(z), true);
  if (z + 1 <= z1) both(ra, z + 1, more(z + 1), true);
  if (z + 2 <= z1) both(rb, z + 2, false, true);
  second(z1 + 1, true);
}

}  // namespace lbm
