// pair_plan.hip -- tile choice for the two-steps-per-pass kernel (host only).
#include <algorithm>
#include <cmath>

#include "pair.hpp"

namespace {

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Addresses of a lattice (no tiles yet); false where the pass does not apply:
// buffer addresses are 32-bit byte offsets and the kernel wraps planes once.
bool set_geometry(PairGeom& g, bool* separable, int q, int nx, int ny, int nz, int px, size_t s,
                  const lbm::PopIndex& L) {
  g.nx = nx;
  g.px = px;
  g.ny = q == 9 ? 1 : ny;
  g.nz = q == 9 ? ny : nz;
  const size_t N = (size_t)px * ny * nz, np = (size_t)px * g.ny;
  const size_t elems = L.bstride ? (size_t)L.bstride * ((N + L.mask) >> L.lb) : (size_t)q * L.pstride;
  if (elems * s >= ((size_t)1 << 32) || g.nz < 4) return false;
  g.bytes = (uint32_t)(elems * s);
  g.pb = L.pstride * (uint32_t)s;
  const int ls = s == 8 ? 3 : (s == 4 ? 2 : 1);
  if (L.bstride) {
    g.sh = (int)L.lb + ls;
    g.kb = (L.bstride - (L.mask + 1)) * (uint32_t)s;
    *separable = np % ((size_t)L.mask + 1) == 0;
    g.zb = (uint32_t)(np / ((size_t)L.mask + 1) * L.bstride * s);
  } else {
    g.sh = 31;
    g.kb = 0;
    *separable = true;
    g.zb = (uint32_t)(np * s);
  }
  return true;
}

// Time of one interval (a plane of every resident work-group) in us, from the
// vector instructions of a CU's waves, its memory traffic and the latency of
// an interval.  The constants are fitted to 3229 timings of splits of 28
// lattices (D3Q19 20 x 16 x 18 to 256^3, D2Q9 64^2 to 2048 x 1024; FP64, FP32
// and FP16): the split they choose is on average 2 % slower than the fastest
// one timed.
struct Model {
  int q;
  size_t s;
  bool masked, big;  // big: the two population buffers exceed what the caches hold

  // resident work-groups of a CU, by registers and LDS
  int per_cu(int columns, bool small) const {
    const size_t lds = (size_t)pair_column_limit(q, s, small) * (2 * q * s + (masked ? 8 : 0));
    return std::max(1, std::min((q == 9 ? 20 : (s == 8 ? 8 : 12)) / ceil_div(columns, 64),
                                (int)(163840 / lds)));
  }
  double interval(int W, int H, int TX, int TY, int px, bool one_tile_wide, double resident) const {
    const double per_wave = 0.087 * (q == 9 ? 0.57 : 1.0) * (masked ? 1.12 : 1.0) *
                            (s == 8 ? 1.59 : (s == 2 ? 1.19 : 1.0));
    // Bytes a row of a tile costs beyond its own: the lines its shifted reads
    // share with the next tile, and those that it writes in part where tiles
    // do not end on lines.  Both cost more in a big lattice (224^3 FP32: tiles
    // 56 wide 486 us a pass, 112 wide 377 us).
    const bool whole_lines = one_tile_wide || ((TX * s) % 128 == 0 && (px * s) % 128 == 0);
    const double shared = big ? 400.0 : 113.0;
    const double partial = whole_lines ? 0.0 : (big ? 300.0 : 86.0);
    const double rate = big ? 50000.0 : 41600.0;  // bytes per us and CU
    const int waves = ceil_div(W * H, 64) + ceil_div(TX * TY, 64);
    const double busy = std::max(per_wave * resident * waves, 0.63);
    const double mem = resident * q * (H * (W * (double)s + shared) + TY * (TX * (double)s + partial)) / rate;
    return 0.46 + std::pow(std::pow(busy, 2.32) + std::pow(mem, 2.32), 1.0 / 2.32);
  }
};

bool is_big(double cells, int q, size_t s) { return 2.0 * cells * q * (double)s > 163e6; }

// Every split of a plane of g into tiles: fn(TX, TY, ntx, nty).
template <typename Fn>
void each_tile(const PairGeom& g, int q, int limit, Fn fn) {
  for (int ntx = 1; ntx <= g.nx; ++ntx) {
    const int TX = ceil_div(g.nx, ntx), W = TX + 2;
    if (TX < 8 && ntx > 1) break;
    const int hmax = q == 9 ? 3 : limit / W;
    if (ceil_div(g.nx, TX) != ntx || W > limit || hmax < 3) continue;
    for (int nty = ceil_div(g.ny, hmax - 2); nty <= g.ny; ++nty) {
      const int TY = ceil_div(g.ny, nty);
      if (ceil_div(g.ny, TY) == nty) fn(TX, TY, ntx, nty);
    }
  }
}

void set_tiles(PairGeom& g, int q, int TX, int TY, int ntx, int nty, int ZC) {
  g.TX = TX;
  g.TY = TY;
  g.W = TX + 2;
  g.H = q == 9 ? 1 : TY + 2;
  g.ntx = ntx;
  g.tiles = ntx * nty;
  g.ZC = ZC;
  g.nblocks = g.tiles * ceil_div(g.nz, ZC);
}

}  // namespace

PairPlan lbm_detail::make_pair_plan(int nx, int ny, int nz, size_t s, bool masked,
                                    const lbm::PopIndex& L, int num_cu) {
  constexpr int q = 19;
  PairPlan best;
  PairGeom g{};
  if (!set_geometry(g, &best.separable, q, nx, ny, nz, nx, s, L)) return best;
  // Cost in us of every split of the lattice into tiles and runs of planes:
  // rounds of work-groups x intervals x the time of an interval.
  const size_t N = (size_t)nx * ny * nz;
  const Model m{q, s, masked, is_big((double)N, q, s)};
  for (bool small : {false, true})
    each_tile(g, q, pair_column_limit(q, s, small), [&](int TX, int TY, int ntx, int nty) {
      const int W = TX + 2, H = TY + 2, per_cu = m.per_cu(W * H, small);
      for (int nzc = 1; nzc <= g.nz; ++nzc) {
        const int ZC = ceil_div(g.nz, nzc);
        if (ceil_div(g.nz, ZC) != nzc) continue;
        const long long blocks = (long long)ntx * nty * nzc;
        if (blocks > 65536) break;
        const long long slots = (long long)num_cu * per_cu;
        const double rounds = (double)((blocks + slots - 1) / slots);
        const double resident = (double)std::min<long long>(per_cu, (blocks + num_cu - 1) / num_cu);
        const double cost = 2.1 + rounds * (ZC + 1.23) * m.interval(W, H, TX, TY, nx, ntx == 1, resident);
        if (cost < best.cost) {
          best.cost = cost;
          best.small = small;
          best.geom = g;
          set_tiles(best.geom, q, TX, TY, ntx, nty, ZC);
        }
      }
    });
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
  if (s != 2)
    best.use = some;
  else if (masked)
    best.use = some && N <= 1100000;
  else
    best.use = some && (N >= 12000000 || (!wave_rows && N <= 1100000));
  return best;
}

// A batch has work-groups enough to fill the card many times over, so a tile is
// judged by the time its work-groups take of a fully occupied CU, each member on
// its own; all members take the larger or all the smaller column limit (the
// 256-box ensemble FP32: 493 us a step with tiles of up to 704 columns, 543 of
// up to 320, 615 in place; 40 boxes of 20-47: 38 / 44 / 43).
//
// 4- and 8-byte storage only: in 16 bits the passes are bound by their
// arithmetic (the ensemble 355 us a step against 308 in place), and the in-place
// kernels' FP16 results round once or twice from cell to cell (v_fma_mixlo), as
// the compiler has it.
PairBatchPlan lbm_detail::make_pair_batch_plan(int q, size_t s, const std::vector<PairMember>& members,
                                               int num_cu) {
  PairBatchPlan plan;
  if (s == 2) return plan;
  double cells = 0.0;
  for (const PairMember& b : members) cells += (double)b.px * b.ny * b.nz;
  const Model m{q, s, false, is_big(cells, q, s)};
  struct Tiled {
    PairGeom geom;
    double interval;  // us of a CU a plane of a tile takes
  };
  std::vector<Tiled> tiled, best;
  double total = 1e300;
  for (bool small : {false, true}) {
    const int limit = pair_column_limit(q, s, small), per_cu = m.per_cu(limit, small);
    double sum = 0.0;
    tiled.clear();
    for (const PairMember& b : members) {
      Tiled t{};
      bool sep = false;
      if (!set_geometry(t.geom, &sep, q, b.nx, b.ny, b.nz, b.px, s, b.pix)) return plan;
      double least = 1e300;
      const PairGeom g = t.geom;
      each_tile(g, q, limit, [&](int TX, int TY, int ntx, int nty) {
        const int W = TX + 2, H = q == 9 ? 1 : TY + 2;
        const double us = m.interval(W, H, TX, TY, b.px, ntx == 1, per_cu) / per_cu;
        if (us * ntx * nty < least) {
          least = us * ntx * nty;
          t.interval = us;
          set_tiles(t.geom, q, TX, TY, ntx, nty, g.nz);
        }
      });
      if (least == 1e300) return plan;
      sum += least * (g.nz + 1.23);
      tiled.push_back(t);
    }
    if (sum < total) {
      total = sum;
      best = tiled;
      plan.small = small;
    }
  }
  // Runs of planes: from one to sixteen to a slot of a work-group, weighing the
  // planes each run repeats against the wait for the last work-groups.
  const int per_cu = m.per_cu(pair_column_limit(q, s, plan.small), plan.small);
  const auto run = [&](const Tiled& t, double target) {
    const int nzc = std::max(1, std::min(t.geom.nz, (int)std::lround(t.geom.nz * t.interval / target)));
    return ceil_div(t.geom.nz, nzc);
  };
  double target = 0.0, least = 1e300;
  for (double d = 1.0; d <= 16.0; d *= 2.0) {
    double work = 0.0, longest = 0.0;
    for (const Tiled& t : best) {
      const int ZC = run(t, total / num_cu / d);
      const double item = (ZC + 1.23) * t.interval;
      work += item * t.geom.tiles * ceil_div(t.geom.nz, ZC);
      longest = std::max(longest, item);
    }
    const double us = work / num_cu + 0.3 * longest * per_cu;
    if (us < least) {
      least = us;
      target = total / num_cu / d;
    }
  }
  // Members go to the XCD with the least work, whole or, the large ones, in
  // eighths (a member of more than a twelfth of the work): neighbouring tiles
  // share one L2 (the 256-box ensemble in FP64, members above a 32nd cut: 832
  // us a step, none cut: 782; three members, none cut: 21.9 against 9.9).  The hardware deals blocks to
  // the XCDs in turn.
  struct Piece {
    int member, first, count;
    double item;  // us of a work-group
  };
  std::vector<Piece> pieces;
  for (size_t k = 0; k < best.size(); ++k) {
    PairGeom& g = best[k].geom;
    g.ZC = run(best[k], target);
    g.nblocks = g.tiles * ceil_div(g.nz, g.ZC);
    const double item = (g.ZC + 1.23) * best[k].interval;
    const int cuts = item * g.nblocks > total / 12.0 ? 8 : 1;
    for (int c = 0; c < cuts; ++c) {
      const int a = (int)((long long)g.nblocks * c / cuts), e = (int)((long long)g.nblocks * (c + 1) / cuts);
      if (e > a) pieces.push_back({(int)k, a, e - a, item});
    }
    plan.threads = std::max(plan.threads, ceil_div(g.W * g.H, 64) * 64);
  }
  std::stable_sort(pieces.begin(), pieces.end(),
                   [](const Piece& a, const Piece& b) { return a.item > b.item; });
  std::vector<PairItem> lists[8];
  double load[8] = {};
  for (const Piece& p : pieces) {
    const int x = (int)(std::min_element(load, load + 8) - load);
    load[x] += p.item * p.count;
    const PairGeom& g = best[p.member].geom;
    for (int id = p.first; id < p.first + p.count; ++id) {
      const int z0 = id / g.tiles * g.ZC;
      lists[x].push_back({g, id % g.tiles, z0, std::min(z0 + g.ZC, g.nz), members[p.member].pop_off,
                          members[p.member].omega});
    }
  }
  size_t rows = 0;
  for (const auto& l : lists) rows = std::max(rows, l.size());
  plan.items.resize(8 * rows);
  for (int x = 0; x < 8; ++x)
    for (size_t r = 0; r < lists[x].size(); ++r) plan.items[8 * r + x] = lists[x][r];
  return plan;
}
