// Host-side device-memory plumbing shared by the library's entry points:
// a buffer record, the allocator in use (the caller's leiden_allocator or
// HIP's stream-ordered allocator) and a process-wide pool of pinned staging
// blocks.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "leiden.h"

namespace lk {

struct DBuf {
  void *p = nullptr;
  size_t cap = 0;
};

constexpr size_t kPinBytes = 65536;

struct ScratchBlock {
  void *p;
  size_t cap;
  int dev;
  uint64_t used;  // number of the call that used it last
};

// Working memory of the stateless calls (leiden_aggregate, leiden_modularity),
// which have no handle to keep it and no caller's allocator.  Mapping it anew
// on each call was most of such a call: R-MAT scale 21, 64M entries, 10 to
// 44 ms for 4 ms of kernels, now 3.8 (a hipMemPool with a release threshold:
// 8.8 ms, it gives most blocks back at each synchronisation).  A call ends by waiting for
// its stream, so its blocks are idle then and any thread and stream of the
// device may use them next.  Kept are at most kScratchKeep bytes and
// kScratchBlocks blocks, none that the last kScratchAge calls left unused;
// all of a device's go when an allocation fails on it (scratch_make_room) or a
// handle is destroyed.
constexpr size_t kScratchKeep = (size_t)2 << 30;
constexpr int kScratchBlocks = 256;
constexpr uint64_t kScratchAge = 16;
struct ScratchCache {
  std::mutex mu;
  ScratchBlock b[kScratchBlocks];
  int n = 0;
  uint64_t calls = 0;
  // the smallest block that holds `want` bytes and at most twice as much
  bool take(int dev, size_t want, ScratchBlock *out) {
    std::lock_guard<std::mutex> lk(mu);
    int best = -1;
    for (int i = 0; i < n; i++)
      if (b[i].dev == dev && b[i].cap >= want && b[i].cap / 2 <= want && (best < 0 || b[i].cap < b[best].cap)) best = i;
    if (best < 0) return false;
    *out = b[best];
    b[best] = b[--n];
    return true;
  }
  // the blocks of an ended call on `dev`, idle; s: a stream of the device to
  // release on
  void give(ScratchBlock *c, int k, int dev, hipStream_t s) {
    std::lock_guard<std::mutex> lk(mu);
    calls++;
    size_t held = 0;
    for (int i = 0; i < n;) {
      if (b[i].dev == dev && b[i].used + kScratchAge < calls) {
        (void)hipFreeAsync(b[i].p, s);
        b[i] = b[--n];
      } else {
        if (b[i].dev == dev) held += b[i].cap;
        i++;
      }
    }
    for (int i = 0; i < k; i++) {
      if (n < kScratchBlocks && c[i].cap <= kScratchKeep - std::min(held, kScratchKeep)) {
        held += c[i].cap;
        b[n] = c[i];
        b[n++].used = calls;
      } else {
        (void)hipFreeAsync(c[i].p, s);
      }
    }
  }
  bool drop(int dev, hipStream_t s) {
    std::lock_guard<std::mutex> lk(mu);
    const int before = n;
    for (int i = 0; i < n;) {
      if (b[i].dev == dev) {
        (void)hipFreeAsync(b[i].p, s);
        b[i] = b[--n];
      } else {
        i++;
      }
    }
    return n < before;
  }
};
inline ScratchCache &scratch_cache() {
  static ScratchCache cache;  // no destructor: calls may run until the process ends
  return cache;
}
inline int stream_device(hipStream_t s) {
  int dev = -1;
  if ((s ? hipStreamGetDevice(s, &dev) : hipGetDevice(&dev)) != hipSuccess) {
    (void)hipGetLastError();
    return -1;
  }
  return dev;
}

// Gives the kept blocks of the stream's device back to the system, for an
// allocation that has failed, a caller's allocator's too.  False when there
// were none, or when the stream is being captured (a release recorded there
// would be made at each replay).
inline bool scratch_make_room(int dev, hipStream_t s) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
  if (cap != hipStreamCaptureStatusNone || !scratch_cache().drop(dev, s)) return false;
  if (hipStreamSynchronize(s) != hipSuccess) return false;
  hipMemPool_t pool;
  if (hipDeviceGetMemPool(&pool, dev) != hipSuccess || hipMemPoolTrimTo(pool, 0) != hipSuccess) (void)hipGetLastError();
  return true;
}

// Device memory of a handle or of a stateless call: obtained from the
// caller's allocator when one is given (leiden_allocator), else from HIP's
// stream-ordered allocator (a stateless call: from its kept blocks first);
// every release is ordered on a stream after the work that last used the
// memory, so no release waits for the device.
struct Alloc {
  leiden_allocator a{};
  bool custom = false;
  bool scratch = false;  // a stateless call: its blocks, released ones too, are listed here until it ends
  int dev = -1;
  int nmine = 0;
  ScratchBlock mine[kScratchBlocks / 2];
  void *raw(size_t bytes, hipStream_t s) {
    void *p = nullptr;
    if (hipMallocAsync(&p, bytes, s) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    return p;
  }
  // *bytes: what is needed, then what the block holds
  void *get(size_t *bytes, hipStream_t s) {
    if (custom) {
      void *p = a.alloc(a.ctx, *bytes, (void *)s);
      if (!p && scratch_make_room(stream_device(s), s)) p = a.alloc(a.ctx, *bytes, (void *)s);
      return p;
    }
    const bool list = scratch && dev >= 0 && nmine < kScratchBlocks / 2;
    ScratchBlock k;
    if (list && scratch_cache().take(dev, *bytes, &k)) {
      mine[nmine++] = k;
      *bytes = k.cap;
      return k.p;
    }
    void *p = raw(*bytes, s);
    if (!p && scratch_make_room(scratch ? dev : stream_device(s), s)) p = raw(*bytes, s);
    if (p && list) mine[nmine++] = ScratchBlock{p, *bytes, dev, 0};
    return p;
  }
  void *get(size_t bytes, hipStream_t s) { return get(&bytes, s); }
  void put(void *p, size_t bytes, hipStream_t s) {
    if (!p) return;
    if (custom) return a.release(a.ctx, p, bytes, (void *)s);
    for (int i = 0; i < nmine; i++)
      if (mine[i].p == p) return;  // see end()
    (void)hipFreeAsync(p, s);
  }
  // end of a stateless call
  void end(hipStream_t s) {
    if (hipStreamSynchronize(s) == hipSuccess) {
      scratch_cache().give(mine, nmine, dev, s);
    } else {
      for (int i = 0; i < nmine; i++) (void)hipFreeAsync(mine[i].p, s);
    }
    nmine = 0;
  }
};

// Pinned host staging blocks (device -> host reads of scalars and small
// arrays) are shared by all handles through a process-wide free list, so that
// releasing a handle never frees pinned memory (which would wait for the
// whole device).
struct PinPool {
  std::mutex mu;
  std::vector<void *> free;
  void *take() {
    {
      std::lock_guard<std::mutex> lk(mu);
      if (!free.empty()) {
        void *p = free.back();
        free.pop_back();
        return p;
      }
    }
    void *p = nullptr;
    if (hipHostMalloc(&p, kPinBytes, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    return p;
  }
  void give(void *p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(mu);
    free.push_back(p);
  }
};
inline PinPool &pin_pool() {
  static PinPool *pool = new PinPool();  // never destroyed: blocks live until the process ends
  return *pool;
}

}  // namespace lk
