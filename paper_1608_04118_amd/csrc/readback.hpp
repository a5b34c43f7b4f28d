// Reading macroscopic fields back to host arrays of doubles.
// Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace ltne {

// A lattice's or batch's hold on the pinned staging memory, which the handles
// of a process share: a readback takes a piece for its duration, up to eight
// pieces are kept for later ones, and the last handle to go frees them.  (A
// piece of its own for each handle would pin 2.4 GB for a hundred of them.)
struct StagingHold {
  StagingHold();
  ~StagingHold();
  StagingHold(const StagingHold&) = delete;
  StagingHold& operator=(const StagingHold&) = delete;
};

// Copies the five fields of n values of elem bytes (4 or 8) that lie one
// after another at device address src to the host arrays outs (nullptr: left
// out), as doubles, after the work on the stream; returns when they are there.
// Arrays that overlap hold the last of their fields, in the order of outs.
// device: the stream's.  The caller's handle has a StagingHold.
hipError_t read_fields(int device, hipStream_t stream, const void* src, int elem, long long n, double* const outs[5]);

}  // namespace ltne
