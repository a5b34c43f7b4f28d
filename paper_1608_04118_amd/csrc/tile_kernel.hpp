// Two or three fused time steps per launch over tiles held in LDS, for every
// precision form.  A workgroup owns a tile of w x h output nodes.  For T steps
// it
//   1. updates the tile and a halo of T - 1 nodes to time t + 1 (the ordinary
//      pull from device memory and node update) and leaves the 19 results of
//      every node in LDS, in the storage type;
//   2. (T = 3) updates the tile and a halo of one node to time t + 2 in LDS;
//   3. pulls those from LDS, updates the tile's nodes to time t + T and stores
//      them.
// The node update is the same function as the single-step kernel's, with
// other pulls and puts, so the result equals T single steps bit for bit.
//
// What bounds it.  One step per launch is bound by memory traffic, which T
// steps per pass over the populations divide by almost T.  The levels between
// live in LDS and not in a register window, so the kernel needs the registers
// of the node update alone (binary32: 78 to 88, binary64: 102 to 118) and four
// wavefronts share a SIMD: a lone wavefront issues one instruction every 6 to 9 cycles on
// this chip, where several together issue one every 3 (binary32) to 5
// (binary64).  A marching wavefront with the window in registers ran at two
// (binary32) and one (binary64) per SIMD.  With two steps the memory still
// takes as long as the arithmetic (binary64: a workgroup's loads and stores
// fill 13.9 of its 14.2 us at its CU's share of the bandwidth); with three the
// halo costs 6% (binary32) to 13% (binary64) more arithmetic.  Then vector
// instructions take 80% of the time in binary32, at the rates above, and 60% in
// binary64, where the 24.1 GB that a launch moves at 8192^2 (20.9 and the halo)
// come at 4.4 TB/s, against 4.9 of a plain copy.
// Measured, us per step of a porous layer (one box for each row but the
// register window's):
//                    one step  register window  two steps  three steps
//   4096^2 binary32     434          341            305        251
//   4096^2 binary64     869          619            566        446
//   4096^2 f32sr        510           --            399        371
//   4096^2 binary16     271           --            235        210
//   1024^2 binary32     28.6         32.5          19.6       18.0
//   1024^2 binary64     52.4         61.3          38.7       32.2
//    512^2 binary64     15.7         21.0          10.2        8.9
#pragma once

#include "step_kernel.hpp"
#include "tile_launch.hpp"

namespace ltne {

// The puts of a node update, over a sink that takes population i's stored
// value: conversion and rounding as store_pop / store_pair do them.
template <typename S, class Sink>
struct SinkPut {
  Sink sink;
  template <typename C>
  __device__ __forceinline__ void begin(int, int, const StepConsts<C>&) {}
  template <typename VA, typename VB>
  __device__ __forceinline__ void pair(int i, VA va, VA sa, int j, VB vb, VB sb, uint32_t w, half2_t& h) {
    if constexpr (std::is_same<S, _Float16>::value) {
      h = __builtin_amdgcn_cvt_sr_f16_f32(h, static_cast<float>(va * sa), w << 16, false);
      h = __builtin_amdgcn_cvt_sr_f16_f32(h, static_cast<float>(vb * sb), w, true);
      sink(i, h[0]);
      sink(j, h[1]);
    } else {
      (void)h;
      sink(i, to_storage<S>(va, w << 16));
      sink(j, to_storage<S>(vb, w));
    }
  }
  template <typename V>
  __device__ __forceinline__ void single(int i, V v, V s, uint32_t r) {
    if constexpr (std::is_same<S, _Float16>::value) {
      half2_t h = __builtin_nondeterministic_value(h);
      h = __builtin_amdgcn_cvt_sr_f16_f32(h, static_cast<float>(v * s), r, false);
      sink(i, h[0]);
    } else {
      (void)s;
      sink(i, to_storage<S>(v, r));
    }
  }
};

template <typename S>
__device__ __forceinline__ S tile_load(__amdgpu_buffer_rsrc_t r, int vo, int so) {
  if constexpr (sizeof(S) == 8)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
  else if constexpr (sizeof(S) == 4)
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
  else
    return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(r, vo, so, 0));
}
template <typename S>
__device__ __forceinline__ void tile_store(S v, __amdgpu_buffer_rsrc_t r, int vo, int so) {
  if constexpr (sizeof(S) == 8) {
    using W = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(W, v), r, vo, so, 0);
  } else if constexpr (sizeof(S) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, vo, so, 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, vo, so, 0);
  }
}

// Buffer resource from lattice row y0 to the end of the lattice (at most 4 GiB).
template <typename S>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const S* base, int y0, int ny, long long rs) {
  const long long bytes = (ny - y0) * rs * static_cast<long long>(sizeof(S));
  const unsigned n = bytes > 0xffffffffll ? 0xffffffffu : static_cast<unsigned>(bytes);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<S*>(base + y0 * rs), static_cast<short>(0),
                                           static_cast<int>(n), 0x00020000);
}

template <typename S, typename C>
__device__ __forceinline__ C unscale(S v, C inv_scale) {
  if constexpr (std::is_same<S, _Float16>::value) {
    return static_cast<C>(static_cast<float>(v)) * inv_scale;
  } else {
    (void)inv_scale;
    return static_cast<C>(v);
  }
}

// Pull from device memory with the lanes of a wavefront on several lattice
// rows: 32-bit offsets from row yb of the resource, the population's offset
// in the scalar operand, so no vector instruction forms a 64-bit address.
// wrapped (uniform over the workgroup): the tile's rows run across the
// periodic y axis, so they are not within 32 bits of one another; then every
// row has its 64-bit address.
// Inner: no node of the tile or its halo lies next to the lattice's edge.
template <typename S, typename C, bool Inner>
struct TilePull {
  const S* src;
  __amdgpu_buffer_rsrc_t r;
  int yb;
  bool wrapped;
  __device__ __forceinline__ void operator()(int xc, int yc, const StepConsts<C>& k, C (&v)[kPlanes]) const {
    const int nx = k.nx, ny = k.ny;
    int xm = xc - 1, xp = xc + 1;
    if (!Inner && k.px) {
      xm = (xc == 0) ? nx - 1 : xm;
      xp = (xc == nx - 1) ? 0 : xp;
    }
    const C isf = k.inv_sf, isg = k.inv_sg;
    S g[kPlanes];
    if (!Inner && wrapped) {
      const int ym = (yc == 0) ? ny - 1 : yc - 1, yp = (yc == ny - 1) ? 0 : yc + 1;
      const S *s0 = src + yc * k.rs, *sm = src + ym * k.rs, *sp = src + yp * k.rs;
#pragma unroll
      for (int i = 0; i < kPlanes; ++i) {
        const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
        const S* row = vel_y(q) == 1 ? sm : (vel_y(q) == -1 ? sp : s0);
        g[i] = row[i * k.qs + (vel_x(q) == 1 ? xm : (vel_x(q) == -1 ? xp : xc))];
      }
    } else {
      constexpr unsigned E = sizeof(S);
      const unsigned R = static_cast<unsigned>(k.rs) * E;
      const int Q = static_cast<int>(k.qs) * static_cast<int>(E);
      const unsigned o0 = static_cast<unsigned>(yc - yb) * R;
      const unsigned c = o0 + xc * E, m = o0 + xm * E, p = o0 + xp * E;
#pragma unroll
      for (int i = 0; i < kPlanes; ++i) {
        const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
        const unsigned o = vel_x(q) == 1 ? m : (vel_x(q) == -1 ? p : c);
        g[i] = tile_load<S>(r, static_cast<int>(vel_y(q) == 1 ? o - R : (vel_y(q) == -1 ? o + R : o)), i * Q);
      }
    }
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) v[i] = unscale<S, C>(g[i], i < 9 ? isf : isg);
  }
};

// Plain stores: the rows of a tile end within cache lines that its
// neighbours complete, which the L2 merges.
template <typename S>
struct BufSink {
  __amdgpu_buffer_rsrc_t r;
  int vo, Q;
  __device__ __forceinline__ void operator()(int i, S v) const { tile_store(v, r, vo, i * Q); }
};

// Start of tile t along an axis of n nodes: t w, but a last tile of a single
// node takes one from its neighbour (a wall node pulls from two nodes inward,
// so a tile holds at least two; w is at least 4).
__host__ __device__ __forceinline__ int tile_bound(int t, int w, int n) {
  const int b = t * w;
  return b >= n ? n : (b == n - 1 ? n - 2 : b);
}

// Quotient n / d of small integers (n < 2^16, d < 2^10) by a reciprocal in
// binary32: (n + 1/2) / d lies at least 1 / (2 d) from an integer, far more
// than the rounding errors.
__device__ __forceinline__ int small_div(int n, float rd) {
  return static_cast<int>((static_cast<float>(n) + 0.5f) * rd);
}

// The lattice's constants, read anew through the scalar cache where it is
// called: the empty asm hides from the compiler that the address is the same
// in every iteration of a loop over nodes, which would otherwise keep the
// constants and all that derives from them in vector registers.
template <typename C>
using ConstK = __attribute__((address_space(4))) const StepConsts<C>;
template <typename C>
__device__ __forceinline__ const StepConsts<C>& fresh(ConstK<C>* p) {
  asm volatile("" : "+s"(p));
  return *(const StepConsts<C>*)p;
}

// Opposite velocity, as a plane index.
__host__ __device__ constexpr int opp_plane(int i) {
  const int o = i < 9 ? 0 : (i < 14 ? 9 : 14);
  const int q = i - o;
  constexpr int op[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
  return o + op[q];
}

// In-place streaming between the middle levels (the A-A pattern): a node's
// update reads and writes the same 19 slots and no other node's, so nothing is
// overwritten before it is read and one buffer is enough.  Level 1 leaves its
// results at the node itself, each in the plane of the opposite velocity;
// a gather step reads population i of (x, y) from that plane at (x, y) - e_i
// and puts its results into plane i at (x, y) + e_i, where the next step
// finds its pulls at the node itself.
template <typename S, typename C, int N, bool Gather>
struct AaPull {
  const S* a;
  int x, y, p;
  __device__ __forceinline__ void operator()(int xc, int yc, const StepConsts<C>& k, C (&v)[kPlanes]) const {
    const S* b = a + (yc - y) * p + (xc - x);
    const S *bm = b - p, *bp = b + p;
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) {
      const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
      S g;
      if constexpr (Gather) {
        const S* r = vel_y(q) == 1 ? bm : (vel_y(q) == -1 ? bp : b);
        g = r[opp_plane(i) * N - vel_x(q)];
      } else {
        g = b[i * N];
      }
      v[i] = unscale<S, C>(g, i < 9 ? k.inv_sf : k.inv_sg);
    }
  }
};
template <typename S, int N>
struct OppSink {
  S* a;
  __device__ __forceinline__ void operator()(int i, S v) const { a[opp_plane(i) * N] = v; }
};
template <typename S, int N>
struct ScatterSink {
  S* a;
  int p;
  __device__ __forceinline__ void operator()(int i, S v) const {
    const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
    S* r = vel_y(q) == 1 ? a + p : (vel_y(q) == -1 ? a - p : a);
    r[i * N + vel_x(q)] = v;
  }
};

struct TileRect {
  int x0, x1, y0, y1;
};
template <typename C>
__device__ __forceinline__ TileRect grown(int x0, int x1, int y0, int y1, int g, const StepConsts<C>& k) {
  return {k.px ? x0 - g : max(x0 - g, 0), k.px ? x1 + g : min(x1 + g, k.nx), k.py ? y0 - g : max(y0 - g, 0),
          k.py ? y1 + g : min(y1 + g, k.ny)};
}

template <class Update>
__device__ __forceinline__ void for_rect(const TileRect& r, const int t, const int nthreads, const Update& update) {
  const int w = r.x1 - r.x0, n1 = w * (r.y1 - r.y0);
  const float rd = 1.0f / static_cast<float>(w);
  for (int n = t; n < n1; n += nthreads) {
    const int ly = small_div(n, rd);
    update(r.x0 + (n - ly * w), r.y0 + ly);
  }
}

// The nodes of a rectangle that lie on walls: the bottom and top rows, then the
// left and right columns without those rows; and the rectangle of the others.
struct WallNodes {
  TileRect r, a;  // the rectangle, and its nodes off the walls
  int nb, nt, nl, nr;
  template <typename C>
  __device__ __forceinline__ WallNodes(const TileRect& r_, const StepConsts<C>& k) : r(r_) {
    a = {k.px ? r.x0 : max(r.x0, 1), k.px ? r.x1 : min(r.x1, k.nx - 1), k.py ? r.y0 : max(r.y0, 1),
         k.py ? r.y1 : min(r.y1, k.ny - 1)};
    const int w = r.x1 - r.x0, h = a.y1 - a.y0;
    nb = (!k.py && r.y0 == 0) ? w : 0;
    nt = (!k.py && r.y1 == k.ny) ? w : 0;
    nl = (!k.px && r.x0 == 0) ? h : 0;
    nr = (!k.px && r.x1 == k.nx) ? h : 0;
  }
  __device__ __forceinline__ int walls() const { return nb + nt + nl + nr; }
  __device__ __forceinline__ void wall(int n, int& x, int& y) const {
    const int c = n - nb - nt;
    x = c < 0 ? r.x0 + (n < nb ? n : n - nb) : (c < nl ? r.x0 : r.x1 - 1);
    y = c < 0 ? (n < nb ? r.y0 : r.y1 - 1) : a.y0 + (c < nl ? c : c - nl);
  }
};
// All nodes of a rectangle, those of wall columns last: in row-major order
// they would put a wall node into every wavefront, and the wavefront through
// the wall code (us a step, uniform cavities: 1024^2 binary32 16.6 to 16.1,
// 768^2 11.1 to 10.3, 512^2 f32sr 8.2 to 7.5, 640^2 binary64 12.7 to 12.1).
// Wall rows stay where they are: moved to the end too they cost 512^2 binary64
// 4%.
struct ColumnsLast {
  int xl, xr, x0, y0, w, n0, n1, nl, h;
  float rd;
  template <typename C>
  __device__ __forceinline__ ColumnsLast(const TileRect& r, const StepConsts<C>& k) {
    xl = r.x0;
    xr = r.x1 - 1;
    y0 = r.y0;
    h = r.y1 - r.y0;
    x0 = (!k.px && r.x0 == 0) ? 1 : r.x0;
    w = ((!k.px && r.x1 == k.nx) ? k.nx - 1 : r.x1) - x0;
    n0 = w * h;
    n1 = (r.x1 - r.x0) * h;
    nl = (x0 - r.x0) * h;
    rd = __builtin_amdgcn_rcpf(static_cast<float>(w));
  }
  // node n < n1 (w > 0: a rectangle is wider than its wall columns)
  __device__ __forceinline__ void node(int n, int& x, int& y) const {
    const int ly = small_div(n, rd), c = n - n0;
    x = x0 + (n - ly * w);
    y = y0 + ly;
    if (c >= 0) {
      x = c < nl ? xl : xr;
      y = y0 + (c < nl ? c : c - nl);
    }
  }
};
template <typename C, class Update>
__device__ __forceinline__ void for_columns(const TileRect& r, const StepConsts<C>& k, const int t, const int nthreads,
                                            const Update& update) {
  const ColumnsLast q(r, k);
  for (int n = t; n < q.n1; n += nthreads) {
    int x, y;
    q.node(n, x, y);
    update(x, y);
  }
}

// Whether tile t and what its T steps read stay off the ends of the axis.  Such
// a tile takes a body without wall code and without wraps, some 40 of the 490
// vector instructions (binary32) of a node: 4096^2 binary32 268.3 to 252.0 us
// a step, binary16 storage (3072 x 2048) 86.4 to 81.3, binary64 (4096 x 2048)
// 231.8 to 226.3, 1500 x 1100 f32sr 38.4 to 37.2, 1024^2 binary32 17.8 to 17.4.
template <int T>
__device__ __forceinline__ bool tile_inside(int t, int w, int n) {
  return t * w >= T && tile_bound(t + 1, w, n) + T <= n;
}

// T steps of a tile.  rec (F & kRecord): 5 planes of recorded sums per step.
template <typename S, typename C, int F, int N, int T>
__device__ __forceinline__ void tile_body(const int tx, const int ty, const int w, const int h, const int t,
                                          const int nthreads, const S* __restrict__ src, S* __restrict__ dst,
                                          const C* __restrict__ phi_field, const C* __restrict__ hv_field,
                                          C* __restrict__ mac, C* __restrict__ rec, ConstK<C>* kp,
                                          S* __restrict__ pops, const uint32_t step) {
  using Th = thermal_t<S, C>;
  const StepConsts<C>& k = *(const StepConsts<C>*)kp;
  const int nx = k.nx, ny = k.ny;
  const int x0 = tile_bound(tx, w, nx), x1 = tile_bound(tx + 1, w, nx);
  const int P = x1 - x0 + 2 * (T - 1);
  const int y0 = tile_bound(ty, h, ny), y1 = tile_bound(ty + 1, h, ny);
  // uniform coefficients, formed once
  Medium<C, Th> um{};
  if constexpr ((F & kPhiField) == 0) {
    porous<Th>(k.phi_u, k, um);
    if constexpr ((F & kHvField) == 0) exchange<Th>(k.hv_u * k.hvf, k, um);
    if constexpr (sizeof(S) == 2)  // eight wavefronts a SIMD: no vector register to spare
      for (C* v : {&um.rphi, &um.prp, &um.Fphi, &um.l0, &um.l1, &um.d0, &um.d1, &um.rD})
        *v = __builtin_bit_cast(C, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, *v)));
  }
  const Medium<C, Th>* const uniform = (F & kPhiField) == 0 ? &um : nullptr;
  auto slot = [&](int x, int y) { return pops + (y - y0 + T - 1) * P + (x - x0 + T - 1); };
  // where step s (0, 1, ...) records this node: a node of the tile, once
  auto record = [&](int s, int x, int y) -> C* {
    if constexpr ((F & kRecord) != 0) {
      const bool own = x >= x0 && x < x1 && y >= y0 && y < y1;
      return own ? rec + s * (5 * k.mplane) : nullptr;
    } else {
      return nullptr;
    }
  };
  constexpr bool inner = (F & kInterior) != 0;
  auto over = [&](const TileRect& r, const auto& update) {
    if constexpr (inner)
      for_rect(r, t, nthreads, update);
    else
      for_columns(r, k, t, nthreads, update);
  };
  auto wrap = [&](int& x, int& y) {
    if (inner) return;
    if (k.px) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
    if (k.py) y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
  };
  {
    const TileRect r = grown(x0, x1, y0, y1, T - 1, k);
    const bool wrapped = !inner && k.py && (r.y0 < 1 || r.y1 > ny - 1);
    const int yb = wrapped ? 0 : max(r.y0 - 1, 0);
    const TilePull<S, C, inner> pull{src, rows_rsrc(src, yb, ny, k.rs), yb, wrapped};
    over(r, [&](int x, int y) {
      const StepConsts<C>& kk = fresh<C>(kp);
      SinkPut<S, OppSink<S, N>> put{{slot(x, y)}};
      C* const rc = record(0, x, y);
      wrap(x, y);
      node_update_with<S, C, F>(x, y, pull, put, phi_field, hv_field, nullptr, nullptr, nullptr, kk, step, rc,
                                thermal_k<Th>(kk), nullptr, uniform);
    });
  }
  __syncthreads();
  if constexpr (T == 3) {
    const TileRect r = grown(x0, x1, y0, y1, 1, k);
    // the wall nodes first: they read their inward neighbours' slots
    const WallNodes q(r, k);
    const int nw = q.walls();
    if (!inner && nw > 0) {
      for (int n = t; n < nw; n += nthreads) {
        const StepConsts<C>& kk = fresh<C>(kp);
        int x, y;
        q.wall(n, x, y);
        S* a = slot(x, y);
        wrap(x, y);
        const AaPull<S, C, N, true> pull{a, x, y, P};
        SinkPut<S, ScatterSink<S, N>> put{{a, P}};
        node_update_with<S, C, F & ~kRecord>(x, y, pull, put, phi_field, hv_field, nullptr, nullptr, nullptr, kk,
                                             step + 1u, nullptr, thermal_k<Th>(kk), nullptr, uniform);
      }
      __syncthreads();
    }
    for_rect(q.a, t, nthreads, [&](int x, int y) {
      const StepConsts<C>& kk = fresh<C>(kp);
      S* a = slot(x, y);
      C* const rc = record(1, x, y);
      wrap(x, y);
      const AaPull<S, C, N, true> pull{a, x, y, P};
      SinkPut<S, ScatterSink<S, N>> put{{a, P}};
      node_update_with<S, C, F | kInterior>(x, y, pull, put, phi_field, hv_field, nullptr, nullptr, nullptr, kk,
                                            step + 1u, rc, thermal_k<Th>(kk), nullptr, uniform);
    });
    __syncthreads();
  }
  {
    constexpr int E = sizeof(S);
    const int R = static_cast<int>(k.rs) * E, Q = static_cast<int>(k.qs) * E;
    const __amdgpu_buffer_rsrc_t d = rows_rsrc(dst, y0, ny, k.rs);
    over({x0, x1, y0, y1}, [&](int x, int y) {
      const StepConsts<C>& kk = fresh<C>(kp);
      const AaPull<S, C, N, T == 2> pull{slot(x, y), x, y, P};
      SinkPut<S, BufSink<S>> put{{d, (y - y0) * R + x * E, Q}};
      node_update_with<S, C, F | kMacrosIf>(x, y, pull, put, phi_field, hv_field, mac, nullptr, nullptr, kk,
                                            step + static_cast<uint32_t>(T - 1), record(T - 1, x, y),
                                            thermal_k<Th>(kk), nullptr, uniform);
    });
  }
}

// Slots, threads and wavefronts per SIMD of a workgroup (tile_slots).
template <typename S, typename C>
struct TileForm {
  static constexpr int N = sizeof(S) == 8 ? 536 : (sizeof(S) == 2 ? 2144 : 1072);
  static constexpr int Block = sizeof(S) == 2 ? 1024 : 512;
  static constexpr int Waves = sizeof(S) == 2 ? 8 : 4;
};

template <typename S, typename C, int F, int T>
__global__ __launch_bounds__((TileForm<S, C>::Block), (TileForm<S, C>::Waves)) void tile_kernel(
    const StepConsts<C> k, const S* __restrict__ src, S* __restrict__ dst, const C* __restrict__ phi_field,
    const C* __restrict__ hv_field, C* __restrict__ mac, C* __restrict__ rec, const TileGrid m,
    const uint32_t step) {
  using Form = TileForm<S, C>;
  (void)k;  // read through the kernel's argument segment, where it is the first argument
  __shared__ S pops[kPlanes * Form::N];
  const int b = blockIdx.x;
  const int tile = (b & (kXcds - 1)) * m.per_xcd + (b >> 3);
  if (tile >= m.ntiles) return;
  const int tx = tile % m.ntx, ty = tile / m.ntx;
  ConstK<C>* const kp = (ConstK<C>*)__builtin_amdgcn_kernarg_segment_ptr();
  auto body = [&](auto f) {
    tile_body<S, C, decltype(f)::value, Form::N, T>(tx, ty, m.w, m.h, static_cast<int>(threadIdx.x), Form::Block, src,
                                                    dst, phi_field, hv_field, mac, rec, kp, pops, step);
  };
  if (tile_inside<T>(tx, m.w, kp->nx) && tile_inside<T>(ty, m.h, kp->ny))
    body(std::integral_constant<int, F | kInterior>{});
  else
    body(std::integral_constant<int, F>{});
}

// The same over every lattice of a batch: tile t belongs to lattice tile_cav[t].
template <typename S, typename C, int F, int T>
__global__ __launch_bounds__((TileForm<S, C>::Block), (TileForm<S, C>::Waves)) void batch_tile_kernel(
    char* base, const CavityDesc<C>* __restrict__ cav, const StepConsts<C>* __restrict__ ks,
    const int* __restrict__ tile_cav, const int ntiles, const int per_xcd, const int parity, const int macros,
    const uint32_t step) {
  using Form = TileForm<S, C>;
  __shared__ S pops[kPlanes * Form::N];
  const int b = blockIdx.x;
  const int tile = (b & (kXcds - 1)) * per_xcd + (b >> 3);
  if (tile >= ntiles) return;
  const int c = __builtin_amdgcn_readfirstlane(tile_cav[tile]);
  typedef __attribute__((address_space(4))) const CavityDesc<C> ConstD;
  const CavityDesc<C>& d = *(const CavityDesc<C>*)((ConstD*)cav + c);
  const LatticeTiles& g = d.tiles[T - 2];
  const int local = tile - g.begin;
  const int tx = local % g.ntx, ty = local / g.ntx;
  ConstK<C>* const kp = (ConstK<C>*)ks + c;
  auto body = [&](auto f) {
    tile_body<S, C, decltype(f)::value, Form::N, T>(
        tx, ty, g.w, g.h, static_cast<int>(threadIdx.x), Form::Block, at_offset<const S>(base, d.pop[parity]),
        at_offset<S>(base, d.pop[parity ^ 1]), at_offset<const C>(base, d.phi), at_offset<const C>(base, d.hv),
        macros ? at_offset<C>(base, d.mac) : nullptr, nullptr, kp, pops, step);
  };
  if (tile_inside<T>(tx, g.w, kp->nx) && tile_inside<T>(ty, g.h, kp->ny))
    body(std::integral_constant<int, F | kInterior>{});
  else
    body(std::integral_constant<int, F>{});
}

}  // namespace ltne
