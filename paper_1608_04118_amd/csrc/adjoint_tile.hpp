// Two steps of the adjoint sweep per launch over tiles held in LDS.
//
// A workgroup owns a tile of w x h nodes.  It sweeps the tile and a halo of
// one node back by one step from device memory, leaves mu of every node in LDS
// and the tile's gradient contributions beside it, then sweeps the tile back
// by the second step and adds both contributions to the gradients, in the
// order of two single sweeps.  The arithmetic is adjoint_node's, so the result
// equals two single sweeps bit for bit.
//
// What bounds it.  A single sweep of the 512^2 adjoint cavity in binary32 takes
// 17 us, of which about 4 are the launch, and its 262144 nodes give each SIMD
// four wavefronts that all start by waiting for memory (212 bytes a node).
// Two steps share the launch, the first wait, and the traffic of mu and of the
// gradients: 31.5 us a launch, that is 15.8 a step (binary64: 64.2 to 41.7 us
// a step of the whole call, with the forward and the recompute).  What is left
// is the wavefronts' chains: about 1050 vector instructions a node, 19
// divisions and 4 square roots among them, behind one another at 4 wavefronts
// a SIMD.  Fewer instructions alone do not help: divisions and square roots
// cut to a third of their instructions left the time as it was.
// The halo of one node costs (w + 2)(h + 2) / w h in work, 1.2 at 32 x 16, one
// of the two fastest shapes (with 64 x 8), two workgroups of 512 threads a CU.
#pragma once

#include "adjoint_kernel.hpp"
#include "tile_kernel.hpp"

namespace ltne {

template <typename Lm, int N>
struct LdsMu {
  const Lm* a;  // slot of node (zx, zy)
  int zx, zy, p;
  __device__ __forceinline__ Lm operator()(int i, int x, int y, int, int, int) const {
    const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
    return a[i * N + (y - zy + vel_y(q)) * p + (x - zx + vel_x(q))];
  }
};

// The nodes of a rectangle without wall nodes: those not next to a wall (one
// lane each), and those next to one (four lanes each, as AdjGrid): row y = 1,
// row y = ny - 2, columns x = 1 and x = nx - 2 without those rows.
struct AdjNodes {
  TileRect r;
  int bx0, by0, bw, nbulk;
  int nrow, c1, ncol;  // nodes of the first row, of both, of a column
  int xl, nedge4;      // the first column, lanes of the nodes next to a wall
  float rd;
  template <typename C>
  __device__ __forceinline__ AdjNodes(const TileRect& r_, const StepConsts<C>& k) : r(r_) {
    const int nx = k.nx, ny = k.ny;
    bx0 = k.px ? r.x0 : max(r.x0, 2);
    by0 = k.py ? r.y0 : max(r.y0, 2);
    bw = max((k.px ? r.x1 : min(r.x1, nx - 2)) - bx0, 0);
    const int bh = max((k.py ? r.y1 : min(r.y1, ny - 2)) - by0, 0);
    nbulk = bw * bh;
    rd = 1.0f / static_cast<float>(max(bw, 1));
    const int rw = max(r.x1 - r.x0, 0);
    const bool low = !k.py && r.y0 <= 1 && r.y1 > 1, high = !k.py && r.y0 <= ny - 2 && r.y1 > ny - 2;
    nrow = low ? rw : 0;
    c1 = nrow + (high ? rw : 0);
    const bool left = !k.px && r.x0 <= 1 && r.x1 > 1, right = !k.px && r.x0 <= nx - 2 && r.x1 > nx - 2;
    ncol = bh;
    xl = left ? 1 : nx - 2;
    nedge4 = 4 * (c1 + ncol * ((left ? 1 : 0) + (right ? 1 : 0)));
  }
  __device__ __forceinline__ void bulk_node(int n, int& x, int& y) const {
    const int ly = small_div(n, rd);
    x = bx0 + (n - ly * bw);
    y = by0 + ly;
  }
  template <typename C>
  __device__ __forceinline__ void edge_node(int e, const StepConsts<C>& k, int& x, int& y) const {
    const int c = e - c1;
    if (c < 0) {
      x = r.x0 + (e < nrow ? e : e - nrow);
      y = e < nrow ? 1 : k.ny - 2;
    } else {
      x = c < ncol ? xl : k.nx - 2;
      y = by0 + (c < ncol ? c : c - ncol);
    }
  }
};

// Calls f(x, y, slot, bulk) for this thread's share of the nodes, bulk a
// true or false type.  The lanes of nodes next to a wall start from the last
// threads, which have the fewest of the others.
template <typename C, class Fn>
__device__ __forceinline__ void for_adj_nodes(const AdjNodes& a, const int t, const int nthreads,
                                              const StepConsts<C>& k, const Fn& f) {
  for (int n = t; n < a.nbulk; n += nthreads) {
    int x, y;
    a.bulk_node(n, x, y);
    f(x, y, 0, std::true_type{});
  }
  for (int n = t ^ (nthreads - 64); n < a.nedge4; n += nthreads) {  // whole wavefronts, the last first
    int x, y;
    a.edge_node(n >> 2, k, x, y);
    f(x, y, n & 3, std::false_type{});
  }
}

// Slots of a workgroup: 19 populations and two gradients a node in half a
// CU's LDS, so two workgroups share a CU.
template <typename Lm>
struct AdjTileForm {
  static constexpr int N = sizeof(Lm) == 8 ? kAdjSlots64 : kAdjSlots32;
  static constexpr int Block = sizeof(Lm) == 8 ? 256 : 512;
  static constexpr int Waves = sizeof(Lm) == 8 ? 2 : 4;
};

template <typename Lm, typename C, typename R>
__global__ __launch_bounds__((AdjTileForm<Lm>::Block), (AdjTileForm<Lm>::Waves)) void adjoint2_kernel(
    const StepConsts<C> k_, const Lm* __restrict__ lam_in, Lm* __restrict__ lam_out, const R* __restrict__ rec1,
    const R* __restrict__ rec0, const R* __restrict__ phi_field, const R* __restrict__ hv_field,
    double* __restrict__ gphi, double* __restrict__ ghv, const TileGrid m, const long long lplane) {
  (void)k_;  // read through the kernel's argument segment, where it is the first argument
  using Form = AdjTileForm<Lm>;
  constexpr int N = Form::N;
  __shared__ Lm mus[kPlanes * N];
  __shared__ double g1[N], h1[N];
  const int b = blockIdx.x;
  const int tile = (b & (kXcds - 1)) * m.per_xcd + (b >> 3);
  if (tile >= m.ntiles) return;
  ConstK<C>* kp = (ConstK<C>*)__builtin_amdgcn_kernarg_segment_ptr();
  const StepConsts<C>& k = *(const StepConsts<C>*)kp;
  const int nx = k.nx, ny = k.ny, t = static_cast<int>(threadIdx.x);
  const int tx = tile % m.ntx, ty = tile / m.ntx;
  const int x0 = tile_bound(tx, m.w, nx), x1 = tile_bound(tx + 1, m.w, nx);
  const int y0 = tile_bound(ty, m.h, ny), y1 = tile_bound(ty + 1, m.h, ny);
  const int P = x1 - x0 + 2;
  auto interior = [&](int g) {
    return TileRect{k.px ? x0 - g : max(x0 - g, 1), k.px ? x1 + g : min(x1 + g, nx - 1),
                    k.py ? y0 - g : max(y0 - g, 1), k.py ? y1 + g : min(y1 + g, ny - 1)};
  };
  {
    const GlobalMu<Lm> mu_in{lam_in, lplane};
    for_adj_nodes(AdjNodes(interior(1), k), t, Form::Block, k, [&](int x, int y, int slot, auto bulk) {
      const StepConsts<C>& kk = fresh<C>(kp);
      const int s = (y - y0 + 1) * P + (x - x0 + 1), o = (y - y0) * (x1 - x0) + (x - x0);
      const bool own = x >= x0 && x < x1 && y >= y0 && y < y1;
      if (k.px) x = wrap1(x, nx);
      if (k.py) y = wrap1(y, ny);
      adjoint_node<Lm, C, R, kAdjStep>(
          bulk, x, y, slot, true, mu_in, rec1, phi_field, hv_field, static_cast<const R*>(nullptr),
          static_cast<const R*>(nullptr), static_cast<const R*>(nullptr), kk,
          [&](int ib, double gp, double gh) {
            if (own) {
              gphi[ib] += gp;
              ghv[ib] += gh;
            }
          },
          [&](int, const Lm (&mu)[19], double gp, double gh, const NodeMacros<C>&, C) {
#pragma unroll
            for (int i = 0; i < kPlanes; ++i) mus[i * N + s] = mu[i];
            if (own) {
              g1[o] = gp;
              h1[o] = gh;
            }
          });
    });
  }
  __syncthreads();
  for_adj_nodes(AdjNodes(interior(0), k), t, Form::Block, k, [&](int x, int y, int slot, auto bulk) {
    const StepConsts<C>& kk = fresh<C>(kp);
    const int s = (y - y0 + 1) * P + (x - x0 + 1), o = (y - y0) * (x1 - x0) + (x - x0);
    adjoint_node<Lm, C, R, kAdjStep>(
        bulk, x, y, slot, true, LdsMu<Lm, N>{mus + s, x, y, P}, rec0, phi_field, hv_field, static_cast<const R*>(nullptr),
        static_cast<const R*>(nullptr), static_cast<const R*>(nullptr), kk,
        [&](int ib, double gp, double gh) {
          gphi[ib] += gp;
          ghv[ib] += gh;
        },
        [&](int iz, const Lm (&mu)[19], double gp, double gh, const NodeMacros<C>&, C) {
#pragma unroll
          for (int i = 0; i < kPlanes; ++i) lam_out[i * lplane + iz] = mu[i];
          gphi[iz] = (gphi[iz] + g1[o]) + gp;
          ghv[iz] = (ghv[iz] + h1[o]) + gh;
        });
  });
}

}  // namespace ltne
