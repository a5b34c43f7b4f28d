// Up to eight fused time steps per launch for small lattices, for every
// precision form, with one thread a node.  A workgroup owns a tile of w x h
// output nodes.  It loads the tile and a halo of nsub nodes into LDS and
// advances them between two LDS buffers, every step one ring less, until the
// tile is left.  The node update is the single-step kernel's with other pulls
// and puts, so the result equals nsub single steps bit for bit.
//
// What bounds it.  A lattice of a few thousand nodes leaves most of the chip
// idle, and a step is the launch, the first loads and one node's chain of some
// 430 instructions, of which a lone wavefront issues one every 5 to 9 cycles.
// More steps a launch divide the first two, at the price of halo nodes that
// idle CUs compute; so at most one tile is given to a CU.  Each step's nodes
// are dealt anew to the threads from the first on, so a shrinking rectangle
// leaves whole wavefronts idle.  Two LDS buffers need one barrier a step and no
// separate pass over wall nodes.  Neighbouring tiles go to the same XCD, whose
// L2 holds the halo that the launch before wrote (192^2 binary64, 12 x 12: 3.9
// us a step with tiles dealt over the XCDs, 3.2 this way).
// Measured against launches of three steps (tile_kernel), us per step:
//            binary64     binary32     binary16     f32sr
//    64^2   3.30  2.09   3.16  2.07   3.63  2.24   3.79  2.39
//   128^2   3.24  2.31   3.02  2.16   3.38  2.35   3.55  2.59
//   192^2   3.65  2.85   3.25  2.41   3.52  2.52   3.71  2.99
//   256^2    --    --    3.55  2.79   3.79  2.84   4.30  3.64
//   320^2    --    --    4.20  3.21   4.20  3.27   5.07  4.34
#pragma once

#include "tile_kernel.hpp"

namespace ltne {

template <typename S, typename C, int N>
struct LdsPull {
  const S* a;  // slot of node (x, y)
  int x, y, p;
  __device__ __forceinline__ void operator()(int xc, int yc, const StepConsts<C>& k, C (&v)[kPlanes]) const {
    const S* b = a + (yc - y) * p + (xc - x);
    const S *bm = b - p, *bp = b + p;
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) {
      const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
      const S* r = vel_y(q) == 1 ? bm : (vel_y(q) == -1 ? bp : b);
      v[i] = unscale<S, C>(r[i * N - vel_x(q)], i < 9 ? k.inv_sf : k.inv_sg);
    }
  }
};
// To LDS, or on the last step to device memory.
template <typename S, int N>
struct SlotSink {
  S* a;
  __device__ __forceinline__ void operator()(int i, S v) const { a[i * N] = v; }
};
template <typename S>
struct RowSink {
  S* a;
  long long qs;
  __device__ __forceinline__ void operator()(int i, S v) const { a[i * qs] = v; }
};

template <typename S, typename C>
struct SmallForm {
  static constexpr int Block = small_slots(sizeof(S), sizeof(C));
};

template <typename S, typename C, int F>
__global__ __launch_bounds__((SmallForm<S, C>::Block)) void small_kernel(
    const StepConsts<C> k_, const S* __restrict__ src, S* __restrict__ dst, const C* __restrict__ phi_field,
    const C* __restrict__ hv_field, C* __restrict__ mac, const TileGrid m, const int nsub, const uint32_t step) {
  (void)k_;  // read through the kernel's argument segment, where it is the first argument
  using Th = thermal_t<S, C>;
  constexpr int N = SmallForm<S, C>::Block;
  constexpr bool has_phi = (F & kPhiField) != 0, has_hv = (F & kHvField) != 0;
  __shared__ S pops[2][kPlanes * N];
  __shared__ C phis[has_phi ? N : 1], hvs[has_hv ? N : 1];
  const StepConsts<C>& k = *(const StepConsts<C>*)(ConstK<C>*)__builtin_amdgcn_kernarg_segment_ptr();
  const int t = static_cast<int>(threadIdx.x), nx = k.nx, ny = k.ny;
  const int b = static_cast<int>(blockIdx.x), tile = (b & (kXcds - 1)) * m.per_xcd + (b >> 3);
  if (tile >= m.ntiles) return;
  const int tx = tile % m.ntx, ty = tile / m.ntx;
  const int x0 = tile_bound(tx, m.w, nx), x1 = tile_bound(tx + 1, m.w, nx);
  const int y0 = tile_bound(ty, m.h, ny), y1 = tile_bound(ty + 1, m.h, ny);
  const TileRect all = grown(x0, x1, y0, y1, nsub, k);
  const int P = all.x1 - all.x0;
  // node t of a rectangle; past the ends of a periodic axis (by at most nsub
  // nodes) it is the node there once wrapped
  auto node = [&](const TileRect& r, int& slot, int& x, int& y) {
    const int w = r.x1 - r.x0;
    const int ly = small_div(t, __builtin_amdgcn_rcpf(static_cast<float>(w)));
    x = r.x0 + (t - ly * w);
    y = r.y0 + ly;
    slot = (y - all.y0) * P + (x - all.x0);
    const bool in = y < r.y1;
    if (k.px) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    if (k.py) y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
    return in;
  };
  int slot, x, y;
  if (node(all, slot, x, y)) {
    const S* a = src + (y * k.rs + x);
    S v[kPlanes];
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) v[i] = a[i * k.qs];
    if constexpr (has_phi) phis[slot] = phi_field[y * nx + x];
    if constexpr (has_hv) hvs[slot] = hv_field[y * nx + x];
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) pops[0][i * N + slot] = v[i];
  }
  Medium<C, Th> um{};
  if constexpr (!has_phi) {
    porous<Th>(k.phi_u, k, um);
    if constexpr (!has_hv) exchange<Th>(k.hv_u * k.hvf, k, um);
  }
  const Medium<C, Th>* const uniform = has_phi ? nullptr : &um;
  auto center = [&]() -> CenterFields<C> {  // of the node that (x, y) pulls
    const int cx = (!k.px && x == 0) ? 1 : ((!k.px && x == nx - 1) ? -1 : 0);
    const int cy = (!k.py && y == 0) ? 1 : ((!k.py && y == ny - 1) ? -1 : 0);
    const int c = slot + cy * P + cx;
    return {has_phi ? phis[has_phi ? c : 0] : k.phi_u, has_hv ? hvs[has_hv ? c : 0] : k.hv_u};
  };
  for (int s = 0; s < nsub - 1; ++s) {
    const bool in = node(grown(x0, x1, y0, y1, nsub - 1 - s, k), slot, x, y);
    __syncthreads();
    if (in) {
      const CenterFields<C> cf = center();
      const LdsPull<S, C, N> pull{pops[s & 1] + slot, x, y, P};
      SinkPut<S, SlotSink<S, N>> put{{pops[(s & 1) ^ 1] + slot}};
      node_update_with<S, C, F>(x, y, pull, put, phi_field, hv_field, nullptr, nullptr, nullptr, k,
                                step + static_cast<uint32_t>(s), nullptr, thermal_k<Th>(k), &cf, uniform);
    }
  }
  const bool in = node({x0, x1, y0, y1}, slot, x, y);
  __syncthreads();
  if (in) {
    const CenterFields<C> cf = center();
    const LdsPull<S, C, N> pull{pops[(nsub - 1) & 1] + slot, x, y, P};
    SinkPut<S, RowSink<S>> put{{dst + (y * k.rs + x), k.qs}};
    node_update_with<S, C, F | kMacrosIf>(x, y, pull, put, phi_field, hv_field, mac, nullptr, nullptr, k,
                                          step + static_cast<uint32_t>(nsub - 1), nullptr, thermal_k<Th>(k), &cf,
                                          uniform);
  }
}

}  // namespace ltne
