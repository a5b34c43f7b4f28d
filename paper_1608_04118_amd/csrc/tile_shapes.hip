// Tile shapes of the launches of several steps, chosen on the host, and the
// dispatch over the precision forms.
#include <algorithm>
#include <map>
#include <utility>
#include <vector>

#include "host_common.hpp"
#include "tile_launch.hpp"

namespace ltne {
namespace {

constexpr int kCus = 256;

int waves(int nodes) { return (nodes + 63) / 64; }
int ceil_div(int a, int b) { return (a + b - 1) / b; }
// Wavefront passes over the nodes of a full tile: the tile and the halo that
// each of the nsub steps needs.
int tile_passes(int w, int h, int nsub) {
  int n = 0;
  for (int g = 0; g < nsub; ++g) n += waves((w + 2 * g) * (h + 2 * g));
  return n;
}

// Whether the kernel can address a tile of h rows of this lattice: byte
// offsets from the first row that it reads stay within 31 bits.
bool rows_fit(const lbm_ltne_params& p, int h) {
  const long long row = kPlanes * pop_row_elems(p.nx) * static_cast<long long>(storage_bytes(p.precision));
  return (h + 2 * kTileSteps) * row < (1LL << 31);
}

TileGrid grid_of(const lbm_ltne_params& p, int w, int h) {
  TileGrid g{};
  g.w = w;
  g.h = h;
  g.ntx = ceil_div(p.nx, w);
  g.ntiles = g.ntx * ceil_div(p.ny, h);
  g.per_xcd = ceil_div(g.ntiles, kXcds);
  return g;
}

// Passes of the busiest CU, which holds ceil(tiles / 256) tiles.
long long busiest_passes(const TileGrid& g, int nsub) {
  return static_cast<long long>(ceil_div(g.ntiles, kCus)) * tile_passes(g.w, g.h, nsub);
}

// The shape with the fewest passes among those that split both axes evenly and
// whose halo of nsub - 1 nodes fits `slots` slots; among equals the widest
// rows.  per_cu: passes of the busiest CU; else of all tiles together.  For each
// width the heights that can be the best are tried: the tallest tiles and the
// next three that give another count.
TileGrid best_shape(const lbm_ltne_params& p, int nsub, int slots, bool per_cu) {
  // the next smaller even split of n nodes than tiles of size s
  auto next = [](int n, int s) { return ceil_div(n, ceil_div(n, s - 1)); };
  const int g2 = 2 * (nsub - 1);
  const int wmax = std::min(256, slots / (4 + g2) - g2);
  TileGrid best{};
  long long least = 0;
  for (int w = p.nx <= wmax ? p.nx : next(p.nx, wmax + 1); w >= 3; w = next(p.nx, w)) {
    const int we = std::max(4, w), ntx = ceil_div(p.nx, we), hmax = slots / (we + g2) - g2;
    int nty = ceil_div(p.ny, hmax);
    for (int tries = 0; tries < 4; ++tries) {
      // the most tiles along y that leave the busiest CU's count as it is
      if (per_cu) nty = std::max(nty, ceil_div(ntx * nty, kCus) * kCus / ntx);
      const int he = std::max(4, ceil_div(p.ny, nty));
      if (rows_fit(p, he)) {
        const TileGrid g = grid_of(p, we, he);
        const long long c = per_cu ? busiest_passes(g, nsub)
                                   : static_cast<long long>(g.ntiles) * tile_passes(we, he, nsub);
        if (best.ntiles == 0 || c < least) {
          best = g;
          least = c;
        }
      }
      if (he == 4) break;
      nty = ceil_div(p.ny, he - 1);
    }
    if (w <= 4) break;
  }
  return best;
}

}  // namespace

// Large lattices (2048 tiles and more, eight per CU) take one shape that ran
// fastest, or within 1% of it, on a layer (us per step, three steps: 4096^2
// binary32 48 x 16: 251, 32 x 24: 255, 64 x 11: 255, 28 x 28: 260; 4096 x 2048
// binary64 24 x 15: 225, 32 x 10: 232, 20 x 18: 233, 16 x 22: 241; 3072^2 f32sr
// 48 x 16: 210, 32 x 24: 208, 64 x 11: 216; 3072 x 2048 binary16 54 x 30: 82,
// 64 x 26: 82, 32 x 52: 84) -- unless that shape leaves so much of its last
// tiles empty that it takes over 4/3 times the passes of the best even split.
// Of 128 large lattices from 24 to 400000 nodes wide, those up to that line ran
// at 0.90 to 1.19 times the even split's time with the one shape, those past it
// at 1.00 to 1.64 (400000 x 6 binary64 126 us a step, 89 with the even split;
// 49 x 40000 f32sr 98, 66; 55 x 40000 binary16 62, 38), and those alone had been
// slower than single steps or a register window (108, 78, 46).  On smaller ones a launch takes 4.2 us plus 0.23 us (binary32)
// times the passes of the busiest CU, which holds ceil(tiles / 256) tiles (two
// steps, checked from 257 x 193 to 1024^2 within 3%): that product is made
// smallest.
TileGrid tile_grid(const lbm_ltne_params& p, int nsub) {
  // by steps and precision
  static const int wide[2][4][2] = {{{32, 13}, {64, 14}, {62, 24}, {48, 16}}, {{24, 15}, {48, 16}, {54, 30}, {48, 16}}};
  const int w = wide[nsub - 2][p.precision][0], h = wide[nsub - 2][p.precision][1];
  const TileGrid even = best_shape(p, nsub, tile_slots(p.precision), true);
  if (p.nx >= w && rows_fit(p, h)) {
    const TileGrid g = grid_of(p, w, h);
    if (g.ntiles >= 8 * kCus && (even.ntiles == 0 || 3 * busiest_passes(g, nsub) <= 4 * busiest_passes(even, nsub)))
      return g;
  }
  return even;
}

// A lattice is small if at most 256 tiles, one a CU, cover it with at least
// four steps a launch (512 nodes a workgroup with their halo in binary64, 960
// to 1024 in the other forms): then every such launch measured beat three steps
// over the larger kernel's tiles, from 48^2 (2.2 against 3.3 us a step in
// binary64, 2.05 against 3.2 in binary32) to the largest (257 x 193 binary64
// 3.4 against 4.0, 256^2 with three steps 4.14 against 4.17; 384^2 binary32 4.0
// against 5.1).  Of the steps and shapes the one with the shortest predicted
// step is taken: a launch takes fixed + T per_step + units per_unit us, where a
// unit is a step's ceil(wavefronts / 4) on the CU's four SIMDs (fitted to 558
// launches from 48^2 to 384^2, 2.8% rms, at most 9%).
SmallTiles small_tiles(const lbm_ltne_params& p) {
  // by precision: fixed, per step, per unit
  static const double cost[4][3] = {{6.26, 0.46, 0.80}, {5.14, 0.73, 0.55}, {4.75, 1.12, 0.44}, {5.99, 0.54, 0.94}};
  const double* c = cost[p.precision];
  const int slots = small_slots(storage_bytes(p.precision), compute_bytes(p.precision));
  SmallTiles best{};
  if (static_cast<long long>(p.nx) * p.ny > static_cast<long long>(kCus) * slots) return best;
  double least = 0.0;
  // a halo wraps round a periodic axis once
  const int tmax = std::min({kSmallSteps, p.periodic_x ? p.nx : kSmallSteps, p.periodic_y ? p.ny : kSmallSteps});
  for (int T = 4; T <= tmax; ++T) {
    for (int ntx = 1; ntx <= kCus; ++ntx) {
      const int w = std::max(4, ceil_div(p.nx, ntx));
      const int nty = kCus / ceil_div(p.nx, w);
      const int h = std::max(4, ceil_div(p.ny, nty));
      if (w + 2 * T <= slots / (4 + 2 * T) && (w + 2 * T) * (h + 2 * T) <= slots) {
        int units = 0;
        for (int g = 0; g < T; ++g)
          units += ceil_div(waves(std::min(w + 2 * g, p.nx) * std::min(h + 2 * g, p.ny)), 4);
        const double us = (c[0] + T * c[1] + units * c[2]) / T;
        if (best.steps == 0 || us < least) {
          best.grid = grid_of(p, w, h);
          best.steps = T;
          least = us;
        }
      }
      if (w == 4) break;
    }
  }
  return best;
}

TileGrid adjoint_tile_grid(const lbm_ltne_params& p, int slots) { return best_shape(p, 2, slots, true); }

// A batch: each lattice takes the shape with the fewest passes in all; the
// largest tile size allowed is the one whose estimate for the whole batch
// (tiles per CU, rounded up, times the mean passes of a tile) is smallest, so
// that a small batch is split finely enough to fill the chip (from eight
// tiles per CU on, smaller ones only add halo nodes).
void tile_batch_grids(int n, const lbm_ltne_params* ps, int nsub, TileGrid* out) {
  double least = -1.0;
  std::vector<TileGrid> g(n);
  for (int slots = tile_slots(ps[0].precision); slots >= 64; slots /= 2) {
    long long tiles = 0, passes = 0;
    bool ok = true;
    std::map<std::pair<int, int>, TileGrid> known;  // lattices of equal size take the same tiles
    for (int i = 0; i < n && ok; ++i) {
      const auto at = known.emplace(std::make_pair(ps[i].nx, ps[i].ny), TileGrid{});
      if (at.second) at.first->second = best_shape(ps[i], nsub, slots, false);
      g[i] = at.first->second;
      ok = g[i].ntiles > 0;
      tiles += g[i].ntiles;
      passes += static_cast<long long>(g[i].ntiles) * tile_passes(g[i].w, g[i].h, nsub);
    }
    if (!ok || tiles > (1LL << 30)) continue;
    const double est = static_cast<double>((tiles + kCus - 1) / kCus) * passes / tiles;
    if (least < 0.0 || est < least) {
      least = est;
      for (int i = 0; i < n; ++i) out[i] = g[i];
    }
    if (tiles >= 8 * kCus) break;
  }
  if (least < 0.0)
    for (int i = 0; i < n; ++i) out[i] = TileGrid{};
}

hipError_t launch_tiles(int precision, const TileLaunch& a) {
  switch (precision) {
    case LBM_FP64: return launch_tiles_f64(a);
    case LBM_FP32: return launch_tiles_f32(a);
    case LBM_FP16S: return launch_tiles_f16s(a);
    default: return launch_tiles_f32sr(a);
  }
}

hipError_t launch_small(int precision, const TileLaunch& a) {
  switch (precision) {
    case LBM_FP64: return launch_small_f64(a);
    case LBM_FP32: return launch_small_f32(a);
    case LBM_FP16S: return launch_small_f16s(a);
    default: return launch_small_f32sr(a);
  }
}

hipError_t launch_batch_tiles(int precision, const BatchTileLaunch& a) {
  switch (precision) {
    case LBM_FP64: return launch_batch_tiles_f64(a);
    case LBM_FP32: return launch_batch_tiles_f32(a);
    case LBM_FP16S: return launch_batch_tiles_f16s(a);
    default: return launch_batch_tiles_f32sr(a);
  }
}

}  // namespace ltne
