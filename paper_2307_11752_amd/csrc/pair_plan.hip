// pair_plan.hip -- tile choice for the two-steps-per-pass kernel (host only).
#include <algorithm>
#include <cmath>

#include "pair.hpp"

namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }

}  // namespace

PairPlan lbm_detail::make_pair_plan(int q, int nx, int ny, int nz, size_t s, bool masked,
                                    const lbm::PopIndex& L, int num_cu) {
  PairPlan best;
  PairGeom g{};
  g.nx = nx;
  g.ny = q == 9 ? 1 : ny;
  g.nz = q == 9 ? ny : nz;
  const size_t N = (size_t)nx * ny * nz, np = (size_t)g.nx * g.ny;
  const size_t elems = L.bstride ? (size_t)L.bstride * ((N + L.mask) >> L.lb) : (size_t)q * L.pstride;
  // buffer addresses are 32-bit byte offsets; the kernel wraps planes once
  if (elems * s >= ((size_t)1 << 32) || g.nz < 4) return best;
  g.bytes = (uint32_t)(elems * s);
  g.pb = L.pstride * (uint32_t)s;
  const int ls = s == 8 ? 3 : (s == 4 ? 2 : 1);
  if (L.bstride) {
    g.sh = (int)L.lb + ls;
    g.kb = (L.bstride - (L.mask + 1)) * (uint32_t)s;
    best.separable = np % ((size_t)L.mask + 1) == 0;
    g.zb = (uint32_t)(np / ((size_t)L.mask + 1) * L.bstride * s);
  } else {
    g.sh = 31;
    g.kb = 0;
    best.separable = true;
    g.zb = (uint32_t)(np * s);
  }
  // Cost in us of every split of the lattice into tiles and runs of planes:
  // rounds of work-groups x intervals x the time of an interval, from the
  // vector instructions of a CU's waves, its memory traffic and the latency of
  // an interval.  The constants are fitted to 3229 timings of splits of 28
  // lattices (D3Q19 20 x 16 x 18 to 256^3, D2Q9 64^2 to 2048 x 1024; FP64, FP32
  // and FP16): the split they choose is on average 2 % slower than the fastest
  // one timed.
  const double per_wave = 0.087 * (q == 9 ? 0.57 : 1.0) * (masked ? 1.12 : 1.0) *
                          (s == 8 ? 1.59 : (s == 2 ? 1.19 : 1.0));
  const bool big = 2.0 * (double)N * q * (double)s > 163e6;
  for (int small = 0; small < 2; ++small) {
    const int limit = pair_column_limit(q, s, small != 0);
    const size_t lds = (size_t)limit * (2 * q * s + (masked ? 8 : 0));
    for (int ntx = 1; ntx <= nx; ++ntx) {
      const int TX = ceil_div(nx, ntx), W = TX + 2;
      if (TX < 8 && ntx > 1) break;
      const int hmax = q == 9 ? 3 : limit / W;
      if (ceil_div(nx, TX) != ntx || W > limit || hmax < 3) continue;
      // Bytes a row of a tile costs beyond its own: the lines its shifted reads
      // share with the next tile, and those that it writes in part where tiles
      // do not end on lines.  Both cost more once the two population buffers
      // exceed what the caches hold (224^3 FP32: tiles 56 wide 486 us a pass,
      // 112 wide 377 us).
      const bool whole_lines = ntx == 1 || ((TX * s) % 128 == 0 && (nx * s) % 128 == 0);
      const double shared = big ? 400.0 : 113.0;
      const double partial = whole_lines ? 0.0 : (big ? 300.0 : 86.0);
      const double rate = big ? 50000.0 : 41600.0;  // bytes per us and CU
      for (int nty = ceil_div(g.ny, hmax - 2); nty <= g.ny; ++nty) {
        const int TY = ceil_div(g.ny, nty), H = q == 9 ? 1 : TY + 2;
        if (ceil_div(g.ny, TY) != nty) continue;
        const int waves = ceil_div(W * H, 64) + ceil_div(TX * TY, 64);
        // resident work-groups of a CU, by registers and LDS
        const int per_cu = std::max(1, std::min((q == 9 ? 20 : (s == 8 ? 8 : 12)) / ceil_div(W * H, 64),
                                                (int)(163840 / lds)));
        for (int nzc = 1; nzc <= g.nz; ++nzc) {
          const int ZC = ceil_div(g.nz, nzc);
          if (ceil_div(g.nz, ZC) != nzc) continue;
          const long long blocks = (long long)ntx * nty * nzc;
          if (blocks > 65536) break;
          const long long slots = (long long)num_cu * per_cu;
          const double rounds = (double)((blocks + slots - 1) / slots);
          const double resident = (double)std::min<long long>(per_cu, (blocks + num_cu - 1) / num_cu);
          const double busy = std::max(per_wave * resident * waves, 0.63);
          const double mem = resident * q * (H * (W * (double)s + shared) + TY * (TX * (double)s + partial)) / rate;
          const double interval = std::pow(std::pow(busy, 2.32) + std::pow(mem, 2.32), 1.0 / 2.32);
          const double cost = 2.1 + rounds * (ZC + 1.23) * (0.46 + interval);
          if (cost < best.cost) {
            best.cost = cost;
            best.small = small != 0;
            g.TX = TX;
            g.TY = TY;
            g.W = W;
            g.H = H;
            g.ntx = ntx;
            g.tiles = ntx * nty;
            g.ZC = ZC;
            g.nblocks = (int)blocks;
            best.geom = g;
          }
        }
      }
    }
  }
  // 4- and 8-byte storage: at every size (us a step in place / two to a pass,
  // FP32 boxes 64^3 12.6 / 6.7, 101 x 77 x 53 14.5 / 11.6, 256^3 389 / 254).
  // 16-bit storage: the passes are bound by their arithmetic, the in-place
  // kernels move half the bytes.  Boxes whose rows the one-wave kernel takes
  // (4 * 2^k <= 256 cells) and up to a million cells stay in place (64^3 5.4 / 5.4, 128^3
  // 23.3 / 25.6), other small boxes do not (80^3 12.0 / 9.6, 101 x 77 x 53 11.5
  // / 8.7); nor do those from 12 million cells on (256^3 189 / 163); with walls,
  // lattices of up to a million cells gain (64^3 10.4 / 8.1, 277 x 95 x 38 30.0
  // / 23.1) and larger ones lose (192^3 103 / 124).
  const bool wave_rows = nx % 4 == 0 && nx <= 256 && ((nx / 4) & (nx / 4 - 1)) == 0;
  const bool some = best.cost < 1e300;
  if (s != 2 || q == 9)
    best.use = some;
  else if (masked)
    best.use = some && N <= 1100000;
  else
    best.use = some && (N >= 12000000 || (!wave_rows && N <= 1100000));
  return best;
}
