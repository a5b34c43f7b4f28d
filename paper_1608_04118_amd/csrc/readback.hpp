// Reading macroscopic fields back to host arrays of doubles.
// Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace ltne {

// Pinned staging memory of one lattice or batch, allocated by the first
// readback: kSlots chunks at most (24 MB in binary64, 12 MB in binary32), no
// more than the fields need.  One user at a time, as the handle that holds it.
struct Staging {
  static constexpr int kSlots = 12;
  char* buf = nullptr;
  size_t bytes = 0;
  hipEvent_t ev[kSlots] = {};
  int nev = 0;
  Staging() = default;
  Staging(const Staging&) = delete;
  Staging& operator=(const Staging&) = delete;
  ~Staging() { release(); }
  void release();
};

// Copies the five fields of n values of elem bytes (4 or 8) that lie one
// after another at device address src to the host arrays outs (nullptr: left
// out), as doubles, after the work on the stream; returns when they are there.
// Arrays that overlap hold the last of their fields, in the order of outs.
// device: the stream's.
hipError_t read_fields(Staging& st, int device, hipStream_t stream, const void* src, int elem, long long n,
                       double* const outs[5]);

}  // namespace ltne
