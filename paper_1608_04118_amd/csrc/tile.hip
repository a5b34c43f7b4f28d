// The tiled kernels (two and three steps, and up to eight of a small lattice)
// of one precision form (LTNE_TILE_FORM, a value of the precision field) and
// their launches.  Compiled once per form, with
// machine-level loop-invariant code motion off: the loop over a workgroup's
// nodes would otherwise keep the binary64 literals of the node update in 46
// vector registers across its iterations (152 registers instead of 110, two
// wavefronts per SIMD instead of four).
#include "small_kernel.hpp"
#include "tile_kernel.hpp"

namespace ltne {

#if LTNE_TILE_FORM == 0
using TS = double;
using TC = double;
#define LTNE_TILE_NAME(f) f##_f64
#elif LTNE_TILE_FORM == 1
using TS = float;
using TC = float;
#define LTNE_TILE_NAME(f) f##_f32
#elif LTNE_TILE_FORM == 2
using TS = _Float16;
using TC = float;
#define LTNE_TILE_NAME(f) f##_f16s
#else
using TS = float;
using TC = double;
#define LTNE_TILE_NAME(f) f##_f32sr
#endif

namespace {

template <int F, int T>
void tiles_ft(const TileLaunch& a) {
  hipLaunchKernelGGL((tile_kernel<TS, TC, F, T>), dim3(kXcds * a.grid.per_xcd), dim3(TileForm<TS, TC>::Block), 0,
                     a.stream, *static_cast<const StepConsts<TC>*>(a.consts), static_cast<const TS*>(a.src),
                     static_cast<TS*>(a.dst), static_cast<const TC*>(a.phi), static_cast<const TC*>(a.hv),
                     static_cast<TC*>(a.mac), static_cast<TC*>(a.rec), a.grid, a.step);
}
template <int F>
void tiles_f(const TileLaunch& a) {
  if constexpr (sizeof(TS) > 2) {  // (no adjoint in binary16 storage)
    if (a.rec) {
      if (a.nsub == 3)
        tiles_ft<F | kRecord, 3>(a);
      else
        tiles_ft<F | kRecord, 2>(a);
      return;
    }
  }
  if (a.nsub == 3)
    tiles_ft<F, 3>(a);
  else
    tiles_ft<F, 2>(a);
}

template <int F>
void small_f(const TileLaunch& a) {
  hipLaunchKernelGGL((small_kernel<TS, TC, F>), dim3(kXcds * a.grid.per_xcd), dim3(SmallForm<TS, TC>::Block), 0, a.stream,
                     *static_cast<const StepConsts<TC>*>(a.consts), static_cast<const TS*>(a.src),
                     static_cast<TS*>(a.dst), static_cast<const TC*>(a.phi), static_cast<const TC*>(a.hv),
                     static_cast<TC*>(a.mac), a.grid, a.nsub, a.step);
}

template <int F, int T>
void batch_tiles_ft(const BatchTileLaunch& a) {
  const int per_xcd = (a.ntiles + kXcds - 1) / kXcds;
  hipLaunchKernelGGL((batch_tile_kernel<TS, TC, F, T>), dim3(kXcds * per_xcd), dim3(TileForm<TS, TC>::Block), 0,
                     a.stream, a.base, static_cast<const CavityDesc<TC>*>(a.cav),
                     static_cast<const StepConsts<TC>*>(a.consts), a.tile_cav, a.ntiles, per_xcd, a.parity,
                     a.macros ? 1 : 0, a.step);
}
template <int F>
void batch_tiles_f(const BatchTileLaunch& a) {
  if (a.nsub == 3)
    batch_tiles_ft<F, 3>(a);
  else
    batch_tiles_ft<F, 2>(a);
}

}  // namespace

hipError_t LTNE_TILE_NAME(launch_tiles)(const TileLaunch& a) {
  switch ((a.phi ? kPhiField : 0) | (a.hv ? kHvField : 0)) {
    case 0: tiles_f<0>(a); break;
    case kPhiField: tiles_f<kPhiField>(a); break;
    case kHvField: tiles_f<kHvField>(a); break;
    default: tiles_f<kPhiField | kHvField>(a);
  }
  return hipGetLastError();
}

hipError_t LTNE_TILE_NAME(launch_small)(const TileLaunch& a) {
  switch ((a.phi ? kPhiField : 0) | (a.hv ? kHvField : 0)) {
    case 0: small_f<0>(a); break;
    case kPhiField: small_f<kPhiField>(a); break;
    case kHvField: small_f<kHvField>(a); break;
    default: small_f<kPhiField | kHvField>(a);
  }
  return hipGetLastError();
}

hipError_t LTNE_TILE_NAME(launch_batch_tiles)(const BatchTileLaunch& a) {
  switch (a.fields) {
    case 0: batch_tiles_f<0>(a); break;
    case kPhiField: batch_tiles_f<kPhiField>(a); break;
    case kHvField: batch_tiles_f<kHvField>(a); break;
    default: batch_tiles_f<kPhiField | kHvField>(a);
  }
  return hipGetLastError();
}

}  // namespace ltne
