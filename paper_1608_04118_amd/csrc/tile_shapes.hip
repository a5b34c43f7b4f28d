// Tile shapes of the two-step launches, chosen on the host, and the dispatch
// over the precision forms.
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
// Wavefront passes over the nodes of a full tile: the tile and its halo to
// t + 1, the tile to t + 2.
int tile_passes(int w, int h) { return waves((w + 2) * (h + 2)) + waves(w * h); }

// Whether the kernel can address a tile of h rows of this lattice: byte
// offsets from the first row that it reads stay within 31 bits.
bool rows_fit(const lbm_ltne_params& p, int h) {
  const long long row = kPlanes * pop_row_elems(p.nx) * static_cast<long long>(storage_bytes(p.precision));
  return (h + 4) * row < (1LL << 31);
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

// The smallest of cost(tiles, passes per tile) over the shapes of at most
// `slots` slots that split an axis evenly; among equals the widest rows.
template <class Cost>
TileGrid best_shape(const lbm_ltne_params& p, int slots, Cost cost) {
  // the next smaller even split of n nodes than tiles of size s
  auto next = [](int n, int s) { return ceil_div(n, ceil_div(n, s - 1)); };
  TileGrid best{};
  double least = 0.0;
  const int wmax = std::min(256, slots / 6 - 2);
  for (int w = p.nx <= wmax ? p.nx : next(p.nx, wmax + 1); w >= 3; w = next(p.nx, w)) {
    const int we = std::max(4, w), hmax = slots / (we + 2) - 2;
    for (int h = p.ny <= hmax ? p.ny : next(p.ny, hmax + 1); h >= 3; h = next(p.ny, h)) {
      const int he = std::max(4, h);
      if (rows_fit(p, he)) {
        const TileGrid g = grid_of(p, we, he);
        const double c = cost(g.ntiles, tile_passes(we, he));
        if (best.ntiles == 0 || c < least) {
          best = g;
          least = c;
        }
      }
      if (h <= 4) break;
    }
    if (w <= 4) break;
  }
  return best;
}

}  // namespace

// Large lattices (2048 tiles and more, eight per CU) take the shape that ran
// fastest on the 4096^2 layer, where long rows save HBM traffic and count for
// more than the fewest halo nodes (binary32 128 x 6: 289 us a step, 64 x 14:
// 295, 32 x 30: 414; binary64 48 x 8: 539, 32 x 13: 546, 16 x 14: 566;
// f32sr 54 x 14: 391, 32 x 28: 395, 64 x 14: 434; binary16 96 x 16: 212,
// 126 x 12: 221).  On smaller ones a launch takes 4.2 us plus 0.23 us
// (binary32) times the passes of the busiest CU, which holds ceil(tiles / 256)
// tiles (checked from 257 x 193 to 1024^2 within 3%): that product is made
// smallest.
TileGrid tile2_grid(const lbm_ltne_params& p) {
  static const int wide[4][2] = {{48, 8}, {128, 6}, {96, 16}, {54, 14}};  // by precision
  const int w = wide[p.precision][0], h = wide[p.precision][1];
  if (p.nx >= w && rows_fit(p, h)) {
    const TileGrid g = grid_of(p, w, h);
    if (g.ntiles >= 8 * kCus) return g;
  }
  return best_shape(p, tile2_slots(p.precision),
                    [](int tiles, int passes) { return static_cast<double>(ceil_div(tiles, kCus)) * passes; });
}

// A batch: each lattice takes the shape with the fewest passes in all; the
// largest tile size allowed is the one whose estimate for the whole batch
// (tiles per CU, rounded up, times the mean passes of a tile) is smallest, so
// that a small batch is split finely enough to fill the chip (from eight
// tiles per CU on, smaller ones only add halo nodes).
void tile2_batch_grids(int n, const lbm_ltne_params* ps, TileGrid* out) {
  double least = -1.0;
  std::vector<TileGrid> g(n);
  for (int slots = tile2_slots(ps[0].precision); slots >= 64; slots /= 2) {
    long long tiles = 0, passes = 0;
    bool ok = true;
    std::map<std::pair<int, int>, TileGrid> known;  // lattices of equal size take the same tiles
    for (int i = 0; i < n && ok; ++i) {
      const auto at = known.emplace(std::make_pair(ps[i].nx, ps[i].ny), TileGrid{});
      if (at.second)
        at.first->second = best_shape(ps[i], slots, [](int t, int c) { return static_cast<double>(t) * c; });
      g[i] = at.first->second;
      ok = g[i].ntiles > 0;
      tiles += g[i].ntiles;
      passes += static_cast<long long>(g[i].ntiles) * tile_passes(g[i].w, g[i].h);
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

hipError_t launch_tile2(int precision, const TileLaunch& a) {
  switch (precision) {
    case LBM_FP64: return launch_tile2_f64(a);
    case LBM_FP32: return launch_tile2_f32(a);
    case LBM_FP16S: return launch_tile2_f16s(a);
    default: return launch_tile2_f32sr(a);
  }
}

hipError_t launch_batch_tile2(int precision, const BatchTileLaunch& a) {
  switch (precision) {
    case LBM_FP64: return launch_batch_tile2_f64(a);
    case LBM_FP32: return launch_batch_tile2_f32(a);
    case LBM_FP16S: return launch_batch_tile2_f16s(a);
    default: return launch_batch_tile2_f32sr(a);
  }
}

}  // namespace ltne
