// Host interface of the tiled kernels (tile_kernel.hpp, small_kernel.hpp,
// adjoint_tile.hpp), which are compiled apart from the rest of the library
// (tile.hip, one object per precision form; adjoint_tile.hip).
#pragma once

#include "common.hpp"
#include "lbm_ltne.h"

namespace ltne {

// Tiles of one lattice of a batch: shape, tiles along x, first entry of the
// lattice in the batch's tile list.
struct LatticeTiles {
  int w, h, ntx, begin;
};

// Buffers of one lattice as byte offsets into the batch's single allocation,
// whose base the kernels take as an argument: addresses formed from a kernel
// argument are known to be global memory, so the loads and stores use a
// scalar base (pointers read from device memory would be generic and turn
// every access into a flat one with a 64-bit per-lane address).
template <typename C>
struct CavityDesc {
  long long pop[2];  // population buffers (storage type), ping-pong
  long long phi;     // per-node porosity, or -1
  long long hv;      // per-node interphase coefficient, or -1
  long long mac;     // macros of the last step (5 planes of nx*ny)
  int tile_begin;    // first entry of this lattice in the combined tile list
  int wave_begin;    // first entry of this lattice in the two-step wavefront list
  int rows2;         // chunk height of its two-step wavefronts
  int pad_;
  LatticeTiles tiles[2];  // of the launches of two and three steps
};

template <typename T>
__device__ __forceinline__ T* at_offset(char* base, long long off) {
  return off < 0 ? nullptr : reinterpret_cast<T*>(base + off);
}

// Most steps of a launch.
constexpr int kTileSteps = 3;

// Tiles of a launch over one lattice.
struct TileGrid {
  int w, h;     // output nodes of a tile; with its halo at most the kernel's slots
  int ntx;      // tiles along x
  int ntiles;   // tiles of the lattice (0: the lattice takes no tiles)
  int per_xcd;  // tiles per XCD; the grid has 8 per_xcd workgroups
};

// LDS slots (nodes) and threads of a workgroup per precision form: two
// workgroups share a CU's 160 KB (19 populations a slot, 81472 bytes a
// workgroup) and its wavefront slots -- 4 wavefronts per SIMD in the forms
// whose node update needs 80 to 128 registers, 8 with binary16 storage (64).
inline int tile_slots(int precision) { return precision == LBM_FP64 ? 536 : (precision == LBM_FP16S ? 2144 : 1072); }

// Threads of a workgroup of the small lattices' kernel, one a node of the tile
// and its halo: two LDS buffers of 19 populations and the two fields in 160 KB.
constexpr int small_slots(int storage_bytes, int compute_bytes) {
  return storage_bytes == 8 ? 512 : (storage_bytes < compute_bytes && compute_bytes == 8 ? 960 : 1024);
}
// Most steps of its launches, and its tiles (steps = 0: the lattice is not small).
constexpr int kSmallSteps = 8;
struct SmallTiles {
  TileGrid grid;
  int steps;
};
SmallTiles small_tiles(const lbm_ltne_params& p);

// The tile shape of one lattice's launches of nsub (2 or 3) steps.
TileGrid tile_grid(const lbm_ltne_params& p, int nsub);
// Tile shapes of a batch's lattices (all of them, or none: ntiles = 0).
void tile_batch_grids(int n, const lbm_ltne_params* ps, int nsub, TileGrid* out);
// Steps of the next launch when left steps remain: three, and two where that
// leaves no single step over.
inline int next_steps(long long left) { return left == 1 ? 1 : (left == 2 || left == 4 ? 2 : 3); }

struct TileLaunch {
  const void* consts;  // StepConsts of the lattice (host)
  const void* src;
  void* dst;
  const void* phi;
  const void* hv;
  void* mac;  // macros of the last step, or nullptr
  void* rec;  // recorded sums of every step (5 planes each), or nullptr (not in binary16 storage)
  TileGrid grid;
  int nsub;       // steps
  uint32_t step;  // number of the first of them
  hipStream_t stream;
};
hipError_t launch_tiles(int precision, const TileLaunch& a);
// The same for a small lattice (a.grid, a.nsub: small_tiles; no rec).
hipError_t launch_small(int precision, const TileLaunch& a);

struct BatchTileLaunch {
  char* base;
  const void* cav;      // CavityDesc of every lattice (device)
  const void* consts;   // StepConsts of every lattice (device)
  const int* tile_cav;  // lattice of every tile (device)
  int ntiles, fields, parity;
  bool macros;
  int nsub;
  uint32_t step;
  hipStream_t stream;
};
hipError_t launch_batch_tiles(int precision, const BatchTileLaunch& a);

// One object of tile.hip per form.
hipError_t launch_tiles_f64(const TileLaunch& a);
hipError_t launch_tiles_f32(const TileLaunch& a);
hipError_t launch_tiles_f16s(const TileLaunch& a);
hipError_t launch_tiles_f32sr(const TileLaunch& a);
hipError_t launch_small_f64(const TileLaunch& a);
hipError_t launch_small_f32(const TileLaunch& a);
hipError_t launch_small_f16s(const TileLaunch& a);
hipError_t launch_small_f32sr(const TileLaunch& a);
hipError_t launch_batch_tiles_f64(const BatchTileLaunch& a);
hipError_t launch_batch_tiles_f32(const BatchTileLaunch& a);
hipError_t launch_batch_tiles_f16s(const BatchTileLaunch& a);
hipError_t launch_batch_tiles_f32sr(const BatchTileLaunch& a);

// Two steps of the adjoint sweep in one launch.  Slots of a workgroup's tile
// and halo: 19 populations and two gradients each in half a CU's LDS.
constexpr int kAdjSlots64 = 480;
constexpr int kAdjSlots32 = 880;
struct Adjoint2Launch {
  const void* consts;  // StepConsts in the sweep's arithmetic type (host)
  const void* lam_in;
  void* lam_out;
  const void* rec1;  // recorded sums of the later step
  const void* rec0;  // and of the one before it
  const void* phi;
  const void* hv;
  double* gphi;
  double* ghv;
  TileGrid grid;
  long long lplane;
  hipStream_t stream;
};
template <typename Lm, typename C, typename R>
hipError_t launch_adjoint2(const Adjoint2Launch& a);
// The tile shape of a lattice's two-step sweeps (slots: one of the above).
TileGrid adjoint_tile_grid(const lbm_ltne_params& p, int slots);

}  // namespace ltne
