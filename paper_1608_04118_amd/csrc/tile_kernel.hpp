// Two fused time steps per launch over tiles held in LDS, for every precision
// form.  A workgroup owns a tile of w x h output nodes.  It
//   1. updates the tile and a halo of one node to time t + 1 (the ordinary
//      pull from device memory and node update) and leaves the 19 results of
//      every node in LDS, in the storage type;
//   2. pulls those from LDS, updates the tile's nodes to time t + 2 and stores
//      them.
// The node update is the same function as the single-step kernel's, with
// other pulls and puts, so the result equals two single steps bit for bit.
//
// What bounds it.  One step per launch is bound by memory traffic, which two
// steps per pass over the populations halve.  The intermediate level lives in
// LDS and not in a register window, so the kernel needs the registers of the
// node update alone (binary32: 83, binary64: 110) and four wavefronts share a
// SIMD: a lone wavefront issues one instruction every 6 to 9 cycles on this
// chip, where several together issue one every 3 (binary32) to 5 (binary64).
// A marching wavefront with the window in registers ran at two (binary32) and
// one (binary64) per SIMD.  Measured, a step of a porous layer, ms:
//                      one step   register window   tiles
//   4096^2 binary32      0.433        0.341         0.289
//   4096^2 binary64      0.869        0.619         0.539
//   4096^2 f32sr         0.510          --          0.391
//   4096^2 binary16      0.271          --          0.212
//   1024^2 binary32      0.0288       0.0325        0.0179
//    512^2 binary64      0.0157       0.0210        0.0093
// The binary32 kernel then issues vector instructions 79% of the cycles and
// moves 4.7 TB/s; the binary64 one moves 5.2 TB/s.
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
template <typename S, typename C>
struct TilePull {
  const S* src;
  __amdgpu_buffer_rsrc_t r;
  int yb;
  bool wrapped;
  __device__ __forceinline__ void operator()(int xc, int yc, const StepConsts<C>& k, C (&v)[kPlanes]) const {
    const int nx = k.nx, ny = k.ny;
    int xm = xc - 1, xp = xc + 1;
    if (k.px) {
      xm = (xc == 0) ? nx - 1 : xm;
      xp = (xc == nx - 1) ? 0 : xp;
    }
    const C isf = k.inv_sf, isg = k.inv_sg;
    S g[kPlanes];
    if (wrapped) {
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

// Pull from the tile in LDS: planes of N slots, rows of p slots; a points at
// the slot of node (x, y), which pulls the populations of (xc, yc).
template <typename S, typename C, int N>
struct LdsTilePull {
  const S* a;
  int x, y, p;
  __device__ __forceinline__ void operator()(int xc, int yc, const StepConsts<C>& k, C (&v)[kPlanes]) const {
    const S* b = a + (yc - y) * p + (xc - x);
    const S *bm = b - p, *bp = b + p;
    const C isf = k.inv_sf, isg = k.inv_sg;
#pragma unroll
    for (int i = 0; i < kPlanes; ++i) {
      const int q = i < 9 ? i : (i < 14 ? i - 9 : i - 14);
      const S* r = vel_y(q) == 1 ? bm : (vel_y(q) == -1 ? bp : b);
      v[i] = unscale<S, C>(r[i * N - vel_x(q)], i < 9 ? isf : isg);
    }
  }
};

template <typename S, int N>
struct LdsSink {
  S* a;
  __device__ __forceinline__ void operator()(int i, S v) const { a[i * N] = v; }
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

template <typename S, typename C, int F, int N>
__device__ __forceinline__ void tile2_body(const int tx, const int ty, const int w, const int h, const int t, const int nthreads,
                                           const S* __restrict__ src, S* __restrict__ dst,
                                           const C* __restrict__ phi_field, const C* __restrict__ hv_field,
                                           C* __restrict__ mac, ConstK<C>* kp, S* __restrict__ pops,
                                           const uint32_t step) {
  using T = thermal_t<S, C>;
  const StepConsts<C>& k = *(const StepConsts<C>*)kp;
  const int nx = k.nx, ny = k.ny;
  const int x0 = tile_bound(tx, w, nx), x1 = tile_bound(tx + 1, w, nx);
  const int P = x1 - x0 + 2;
  const int y0 = tile_bound(ty, h, ny), y1 = tile_bound(ty + 1, h, ny);
  {
    const int rx0 = k.px ? x0 - 1 : max(x0 - 1, 0), rx1 = k.px ? x1 + 1 : min(x1 + 1, nx);
    const int ry0 = k.py ? y0 - 1 : max(y0 - 1, 0), ry1 = k.py ? y1 + 1 : min(y1 + 1, ny);
    const int rw = rx1 - rx0, n1 = rw * (ry1 - ry0);
    const float rd = 1.0f / static_cast<float>(rw);
    const bool wrapped = k.py && (ry0 < 1 || ry1 > ny - 1);
    const int yb = wrapped ? 0 : max(ry0 - 1, 0);
    const TilePull<S, C> pull{src, rows_rsrc(src, yb, ny, k.rs), yb, wrapped};
    for (int n = t; n < n1; n += nthreads) {
      const StepConsts<C>& kk = fresh<C>(kp);
      const int ly = small_div(n, rd), lx = n - ly * rw;
      int x = rx0 + lx, y = ry0 + ly;
      S* slot = pops + (y - y0 + 1) * P + (x - x0 + 1);
      if (k.px) x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
      if (k.py) y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
      SinkPut<S, LdsSink<S, N>> put{{slot}};
      node_update_with<S, C, F>(x, y, pull, put, phi_field, hv_field, nullptr, nullptr, nullptr, kk, step,
                                           nullptr, thermal_k<T>(kk));
    }
  }
  __syncthreads();
  {
    const int ow = x1 - x0, n2 = ow * (y1 - y0);
    const float rd = 1.0f / static_cast<float>(ow);
    constexpr int E = sizeof(S);
    const int R = static_cast<int>(k.rs) * E, Q = static_cast<int>(k.qs) * E;
    const __amdgpu_buffer_rsrc_t r = rows_rsrc(dst, y0, ny, k.rs);
    for (int n = t; n < n2; n += nthreads) {
      const StepConsts<C>& kk = fresh<C>(kp);
      const int ly = small_div(n, rd), lx = n - ly * ow;
      const int x = x0 + lx, y = y0 + ly;
      const LdsTilePull<S, C, N> pull{pops + (ly + 1) * P + lx + 1, x, y, P};
      SinkPut<S, BufSink<S>> put{{r, ly * R + x * E, Q}};
      node_update_with<S, C, F | kMacrosIf>(x, y, pull, put, phi_field, hv_field, mac, nullptr, nullptr, kk, step + 1u, nullptr,
                                thermal_k<T>(kk));
    }
  }
}

// Slots, threads and wavefronts per SIMD of a workgroup (tile2_slots).
template <typename S, typename C>
struct TileForm {
  static constexpr int N = sizeof(S) == 8 ? 536 : (sizeof(S) == 2 ? 2144 : 1072);
  static constexpr int Block = sizeof(S) == 2 ? 1024 : 512;
  static constexpr int Waves = sizeof(S) == 2 ? 8 : 4;
};

template <typename S, typename C, int F>
__global__ __launch_bounds__((TileForm<S, C>::Block), (TileForm<S, C>::Waves)) void tile2_kernel(
    const StepConsts<C> k, const S* __restrict__ src, S* __restrict__ dst, const C* __restrict__ phi_field,
    const C* __restrict__ hv_field, C* __restrict__ mac, const TileGrid m, const uint32_t step) {
  using Form = TileForm<S, C>;
  (void)k;  // read through the kernel's argument segment, where it is the first argument
  __shared__ S pops[kPlanes * Form::N];
  const int b = blockIdx.x;
  const int tile = (b & (kXcds - 1)) * m.per_xcd + (b >> 3);
  if (tile >= m.ntiles) return;
  tile2_body<S, C, F, Form::N>(tile % m.ntx, tile / m.ntx, m.w, m.h, static_cast<int>(threadIdx.x), Form::Block, src,
                               dst, phi_field, hv_field, mac, (ConstK<C>*)__builtin_amdgcn_kernarg_segment_ptr(),
                               pops, step);
}

// The same over every lattice of a batch: tile t belongs to lattice tile_cav[t].
template <typename S, typename C, int F>
__global__ __launch_bounds__((TileForm<S, C>::Block), (TileForm<S, C>::Waves)) void batch_tile2_kernel(
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
  const int local = tile - d.tile2_begin;
  tile2_body<S, C, F, Form::N>(local % d.tile2_ntx, local / d.tile2_ntx, d.tile2_w, d.tile2_h,
                               static_cast<int>(threadIdx.x), Form::Block, at_offset<const S>(base, d.pop[parity]),
                               at_offset<S>(base, d.pop[parity ^ 1]), at_offset<const C>(base, d.phi),
                               at_offset<const C>(base, d.hv), macros ? at_offset<C>(base, d.mac) : nullptr,
                               (ConstK<C>*)ks + c, pops, step);
}

}  // namespace ltne
