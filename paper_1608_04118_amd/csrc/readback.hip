// Reading macroscopic fields back: device memory -> pinned staging -> the
// caller's arrays.
//
// What bounds it.  The arrays are the caller's, usually new, so their pages
// are first touched here: one thread reaches 8 to 14 GB/s of doubles with
// 4 KiB and 2 MiB pages, while the copy engine fills pinned memory at
// 57 GB/s.  A copy straight into pageable memory runs at 9.9 GB/s (18 where
// the pages exist).  So the copy engine goes through a ring of pinned chunks,
// and up to 8 threads move the chunks on, converting binary32 on the way.
// A 4096^2 binary32 lattice (671 MB of doubles): 72 ms with one pageable copy
// and one conversion loop per field, 11 now.
#include "readback.hpp"

#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <type_traits>
#include <utility>
#include <vector>

namespace ltne {

namespace {

#ifndef MADV_POPULATE_WRITE
#define MADV_POPULATE_WRITE 23  // Linux 5.14
#endif

// Doubles that a chunk becomes: 2 MiB, the large page that two threads had
// better not touch first at the same time (chunks end at its multiples).
constexpr long long kChunk = 262144;
// Output bytes that pay for one more thread (starting it takes about 12 us).
constexpr long long kBytesPerThread = 4LL << 20;
constexpr int kMaxThreads = 8;
// Fields up to this size are not worth pinned memory of their own: getting and
// freeing it takes 50 us, and a pageable copy reads 160 KB in 24 us against 23,
// 500 KB in 50 against 43.
constexpr size_t kPageable = 512 << 10;

// Pinned chunks in flight of one readback, and their events: 24 MB at most in
// binary64, 12 MB in binary32, no more than the fields that it has read need.
struct Staging {
  static constexpr int kSlots = 12;
  const int device;
  char* buf = nullptr;
  size_t bytes = 0;
  hipEvent_t ev[kSlots] = {};
  int nev = 0;
  explicit Staging(int d) : device(d) {}
  Staging(const Staging&) = delete;
  Staging& operator=(const Staging&) = delete;
  ~Staging() {
    for (int i = 0; i < nev; ++i) (void)hipEventDestroy(ev[i]);
    if (buf) (void)hipHostFree(buf);
  }
};

// As many as threads that read at the same time are likely to be.
constexpr int kKeptStagings = 8;

// The process's pieces that no readback uses, and the handles alive.  Nothing
// is left to do when the process ends (a handle never closed leaves its memory
// to the system, as its device memory).
struct StagingPool {
  std::mutex m;
  Staging* kept[kKeptStagings] = {};
  int nkept = 0;
  long long handles = 0;
} g_pool;
static_assert(std::is_trivially_destructible<StagingPool>::value, "used by handles closed at the end of the process");

// A piece on the device, of `least` bytes where one is kept, else any or none.
std::unique_ptr<Staging> take_staging(int device, size_t least) {
  std::lock_guard<std::mutex> lock(g_pool.m);
  int at = -1;
  for (int i = 0; i < g_pool.nkept; ++i)
    if (g_pool.kept[i]->device == device && (at < 0 || g_pool.kept[at]->bytes < least)) at = i;
  if (at < 0) return nullptr;
  std::unique_ptr<Staging> s(g_pool.kept[at]);
  g_pool.kept[at] = g_pool.kept[--g_pool.nkept];
  return s;
}

// Back after a readback (no copy into it is in flight).
void keep_staging(std::unique_ptr<Staging> s) {
  std::lock_guard<std::mutex> lock(g_pool.m);
  if (s && s->bytes > 0 && g_pool.nkept < kKeptStagings) g_pool.kept[g_pool.nkept++] = s.release();
}

struct Run {  // `count` values from value `at` of the fields on
  long long at, count;
};

// Gives the whole pages of [p, p + bytes) memory in one call instead of one
// fault at a time while they are written: 0.9 MB of binary32 into 1.8 MB of
// new 4 KiB pages takes 188 us instead of 273.  Where the last page is there
// already the others are taken to be (asking for them all would cost 37 ns a
// page); a kernel that refuses leaves the faults to the writes.
void touch(void* p, size_t bytes) {
  constexpr size_t page = 4096, least = 16 * page;
  const size_t lo = (reinterpret_cast<size_t>(p) + page - 1) & ~(page - 1);
  const size_t hi = (reinterpret_cast<size_t>(p) + bytes) & ~(page - 1);
  unsigned char in = 0;
  if (hi < lo + least || mincore(reinterpret_cast<void*>(hi - page), page, &in) != 0 || (in & 1)) return;
  (void)madvise(reinterpret_cast<void*>(lo), hi - lo, MADV_POPULATE_WRITE);
}

// Moves one chunk from pinned memory to the fields' arrays.
void deliver(const char* from, const Run& r, int elem, long long n, double* const outs[5], bool alone) {
  long long at = r.at, left = r.count;
  while (left > 0) {
    const int f = static_cast<int>(at / n);
    const long long o = at - f * n, c = std::min(left, n - o);
    double* const to = outs[f] + o;
    if (alone) touch(to, static_cast<size_t>(c) * 8);
    if (elem == 8) {
      std::memcpy(to, from, static_cast<size_t>(c) * 8);
    } else {
      const float* s = reinterpret_cast<const float*>(from);
      for (long long i = 0; i < c; ++i) to[i] = s[i];
    }
    from += c * elem;
    at += c;
    left -= c;
  }
}

// The chunks: neighbouring fields in one while they are small; larger fields
// are cut where the array crosses a large page.
void cut(std::vector<Run>& runs, long long n, double* const outs[5]) {
  for (int f = 0; f < 5; ++f) {
    if (!outs[f]) continue;
    long long o = 0;
    while (o < n) {
      const long long past = (reinterpret_cast<size_t>(outs[f] + o) & (kChunk * 8 - 1)) / 8;
      const long long c = std::min(n - o, n > kChunk ? kChunk - past : kChunk);
      const long long at = f * n + o;
      if (n <= kChunk && !runs.empty() && runs.back().at + runs.back().count == at && runs.back().count + c <= kChunk)
        runs.back().count += c;
      else
        runs.push_back(Run{at, c});
      o += c;
    }
  }
}

// Staging memory and events of `nslots` chunks in flight.
hipError_t reserve(Staging& st, size_t bytes, int nslots) {
  const int nev = nslots > 1 ? nslots : 0;
  if (st.bytes >= bytes && st.nev >= nev) return hipSuccess;
  int before = 0;
  hipError_t e = hipGetDevice(&before);
  if (e == hipSuccess && before != st.device) e = hipSetDevice(st.device);  // the events' device
  // an allocation leaves a stream capture elsewhere in the process alone
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (e == hipSuccess) e = hipThreadExchangeStreamCaptureMode(&mode);
  if (e != hipSuccess) return e;
  if (st.bytes < bytes) {
    if (st.buf) (void)hipHostFree(st.buf);
    st.buf = nullptr;
    st.bytes = 0;
    void* p = nullptr;
    e = hipHostMalloc(&p, bytes, hipHostMallocPortable);
    if (e == hipSuccess) {
      st.buf = static_cast<char*>(p);
      st.bytes = bytes;
    }
  }
  while (e == hipSuccess && st.nev < nev) {
    e = hipEventCreateWithFlags(&st.ev[st.nev], hipEventDisableTiming);
    if (e == hipSuccess) ++st.nev;
  }
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (before != st.device) (void)hipSetDevice(before);
  return e;
}

// Whether two fields go to overlapping arrays: then they are delivered one
// after the other, so that what is left there is the last field's.
bool overlapping(long long n, double* const outs[5]) {
  for (int f = 0; f < 5; ++f)
    for (int g = 0; g < f; ++g)
      if (outs[f] && outs[g] && outs[f] < outs[g] + n && outs[g] < outs[f] + n) return true;
  return false;
}

// One pageable copy per field, in their order.
hipError_t read_pageable(hipStream_t stream, const char* src, int elem, long long n, double* const outs[5]) {
  for (int f = 0; f < 5; ++f) {
    if (!outs[f]) continue;
    // binary32 lands in the upper half of the array and is widened in place
    char* const to = reinterpret_cast<char*>(outs[f]) + (elem == 8 ? 0 : n * 4);
    hipError_t e = hipMemcpyAsync(to, src + f * n * elem, n * elem, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return e;
    for (long long i = 0; elem == 4 && i < n; ++i) {
      float v;
      std::memcpy(&v, to + 4 * i, 4);
      const double w = v;
      std::memcpy(outs[f] + i, &w, 8);
    }
  }
  return hipSuccess;
}

}  // namespace

StagingHold::StagingHold() {
  std::lock_guard<std::mutex> lock(g_pool.m);
  ++g_pool.handles;
}

StagingHold::~StagingHold() {
  Staging* last[kKeptStagings];
  int n = 0;
  {
    std::lock_guard<std::mutex> lock(g_pool.m);
    if (--g_pool.handles == 0) {
      n = g_pool.nkept;
      std::copy(g_pool.kept, g_pool.kept + n, last);
      g_pool.nkept = 0;
    }
  }
  for (int i = 0; i < n; ++i) delete last[i];
}

hipError_t read_fields(int device, hipStream_t stream, const void* src_, int elem, long long n,
                       double* const outs[5]) {
  const char* const src = static_cast<const char*>(src_);
  if (overlapping(n, outs)) return read_pageable(stream, src, elem, n, outs);
  std::vector<Run> runs;
  std::vector<std::thread> threads;
  try {
    cut(runs, n, outs);
    threads.reserve(kMaxThreads);
  } catch (const std::bad_alloc&) {
    return hipErrorOutOfMemory;
  }
  const int nruns = static_cast<int>(runs.size());
  if (nruns == 0) return hipSuccess;
  const int nslots = std::min(nruns, Staging::kSlots);
  const size_t slot = static_cast<size_t>(nruns == 1 ? runs[0].count : kChunk) * elem;
  std::unique_ptr<Staging> held = take_staging(device, slot * nslots);
  if (nruns == 1 && slot <= kPageable && (!held || held->bytes < slot)) {
    keep_staging(std::move(held));
    std::unique_ptr<char[]> tmp(new (std::nothrow) char[slot]);
    if (!tmp) return hipErrorOutOfMemory;
    hipError_t e = hipMemcpyAsync(tmp.get(), src + runs[0].at * elem, slot, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e == hipSuccess) deliver(tmp.get(), runs[0], elem, n, outs, true);
    return e;
  }
  if (!held) held.reset(new (std::nothrow) Staging(device));
  if (!held || reserve(*held, slot * nslots, nslots) != hipSuccess) {
    (void)hipGetLastError();
    held.reset();
    return read_pageable(stream, src, elem, n, outs);
  }
  Staging& st = *held;
  auto slot_of = [&](int c) { return st.buf + (c % nslots) * slot; };
  auto send = [&](int c) {
    hipError_t e = hipMemcpyAsync(slot_of(c), src + runs[c].at * elem, runs[c].count * elem, hipMemcpyDeviceToHost,
                                  stream);
    return e == hipSuccess && nruns > 1 ? hipEventRecord(st.ev[c % nslots], stream) : e;
  };
  if (nruns == 1) {
    hipError_t e = send(0);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return e;
    deliver(slot_of(0), runs[0], elem, n, outs, true);
    keep_staging(std::move(held));
    return e;
  }

  long long total = 0;
  for (const Run& r : runs) total += r.count;
  const long long want = std::min<long long>({kMaxThreads, std::max(1u, std::thread::hardware_concurrency()) / 2,
                                              nruns, total * 8 / kBytesPerThread});
  std::atomic<int> arrived{0}, next{0};     // chunks in pinned memory, chunks taken
  std::atomic<int> freed[Staging::kSlots];  // the chunk that may be sent to the slot next
  for (int i = 0; i < Staging::kSlots; ++i) freed[i].store(i, std::memory_order_relaxed);
  auto take = [&](int c) {
    deliver(slot_of(c), runs[c], elem, n, outs, want <= 1);
    freed[c % nslots].store(c + nslots, std::memory_order_release);
  };
  auto work = [&] {
    for (int c; (c = next.fetch_add(1, std::memory_order_relaxed)) < nruns;) {
      int a;
      while ((a = arrived.load(std::memory_order_acquire)) <= c && a >= 0) std::this_thread::yield();
      if (a < 0) return;  // a copy failed
      take(c);
    }
  };
  hipError_t e = hipSuccess;
  int sent = 0;
  for (; sent < nslots && e == hipSuccess; ++sent) e = send(sent);
  if (e == hipSuccess) e = hipEventSynchronize(st.ev[0]);  // the steps before are done; threads that wait spin
  try {
    while (e == hipSuccess && want > 1 && static_cast<long long>(threads.size()) < want) threads.emplace_back(work);
  } catch (const std::exception&) {  // fewer threads
  }
  for (int c = 0; c < nruns && e == hipSuccess; ++c) {
    e = hipEventSynchronize(st.ev[c % nslots]);
    if (e != hipSuccess) break;
    if (threads.empty())
      take(c);
    else
      arrived.store(c + 1, std::memory_order_release);
    // send on whatever slots are free; wait only where nothing else is in flight
    while (sent < nruns && sent <= c + nslots && e == hipSuccess) {
      const bool idle = sent == c + 1;
      if (freed[sent % nslots].load(std::memory_order_acquire) != sent) {
        if (!idle) break;
        std::this_thread::yield();
        continue;
      }
      e = send(sent);
      ++sent;
    }
  }
  if (e != hipSuccess) arrived.store(-1, std::memory_order_release);
  for (std::thread& t : threads) t.join();
  if (e != hipSuccess)
    (void)hipStreamSynchronize(stream);  // no copy into the staging memory is left
  else
    keep_staging(std::move(held));
  return e;
}

}  // namespace ltne
