// Device memory of the library (host code): hipMalloc behind a bounded pool of
// idle blocks.
//
// The one-shot entry points (Gamma, single-shot conductivity, time evolution,
// reconstructions, one-shot DOS) allocate their workspace on each call.  Memory
// that has been written once costs the driver about 23 ms per GB to hand out
// again: a 512 x 512 spinful Gamma call (17 GB of Chebyshev blocks, 27 ms of
// kernels) took 0.5 s, a 0.5 GB one (2.6 ms of kernels) 15 ms.  Released blocks
// are therefore kept for later calls, within these bounds:
// - per device, idle blocks take at most an eighth of its memory, and a block is
//   kept only while at least as much as all idle blocks stays free for others;
//   the oldest go first.  Every release is held against the bound; the free memory
//   in it is read again after each 16 MB released (the query takes longer than the
//   rest of a small release);
// - per device, at most 1024 idle blocks (a request looks at each);
// - an allocation that fails gives every idle block back and tries once more;
// - kpm_release_workspace() gives them back on request;
// - a block serves a request only if it is at most an eighth larger (or 64 KB).
// Only blocks whose caller has waited for its work become idle, so that they may be
// used on any stream at once; those of a call that failed before or in its wait go
// through hipFree, which waits.  The pool itself never synchronises: a device-wide
// wait fails, and invalidates the capture, while any thread captures a stream.
// One mutex covers the bookkeeping; blocks in use by different threads are
// distinct.

#include "kpm_internal.h"

#include <algorithm>
#include <list>
#include <mutex>
#include <unordered_map>

namespace kpm {

namespace {

constexpr size_t kLookEvery = size_t(16) << 20;
constexpr size_t kMaxIdle = 1024;

struct Block {
  void* p;
  size_t cap;
  int dev;
};

// The idle blocks of one device.
struct Idle {
  size_t bytes = 0, count = 0;
  size_t bound = 0;                          // on bytes, from the last look at the device's memory
  size_t unseen = kLookEvery;                // bytes released since
};

struct Pool {
  std::mutex mu;
  std::unordered_map<void*, Block> used;
  std::list<Block> idle;                        // oldest first
  std::unordered_map<int, Idle> idle_of;
};

// Never destroyed: objects with static lifetime may still release memory at exit.
Pool& pool() {
  static Pool* p = new Pool();
  return *p;
}

size_t round_up(size_t bytes) {
  const size_t g = bytes < (size_t(1) << 20) ? size_t(4) << 10 : size_t(2) << 20;
  return (std::max<size_t>(bytes, 1) + g - 1) / g * g;
}

std::list<Block>::iterator drop(Pool& P, std::list<Block>::iterator it) {
  Idle& d = P.idle_of[it->dev];
  d.bytes -= it->cap;
  d.count -= 1;
  return P.idle.erase(it);
}

// Gives back idle blocks of a device, oldest first, until at most keep bytes and
// count blocks are left.
size_t trim(Pool& P, int dev, size_t keep, size_t count) {
  const Idle& d = P.idle_of[dev];
  size_t gone = 0;
  for (auto it = P.idle.begin(); it != P.idle.end() && (d.bytes > keep || d.count > count);) {
    if (it->dev != dev) {
      ++it;
      continue;
    }
    gone += it->cap;
    (void)hipFree(it->p);
    it = drop(P, it);
  }
  return gone;
}

}  // namespace

hipError_t pool_malloc(void** out, size_t bytes) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const size_t need = round_up(bytes);
  try {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto best = P.idle.end();
    for (auto it = P.idle.begin(); it != P.idle.end(); ++it)
      if (it->dev == dev && it->cap >= need && it->cap - need <= std::max(need / 8, size_t(64) << 10) &&
          (best == P.idle.end() || it->cap < best->cap))
        best = it;
    if (best != P.idle.end()) {
      P.used.emplace(best->p, *best);
      *out = best->p;
      drop(P, best);
      return hipSuccess;
    }
    void* p = nullptr;
    e = hipMalloc(&p, need);
    if (e == hipErrorOutOfMemory && trim(P, dev, 0, 0) > 0) {
      (void)hipGetLastError();
      e = hipMalloc(&p, need);
    }
    if (e != hipSuccess) return e;
    try {
      P.used.emplace(p, Block{p, need, dev});
    } catch (...) {
      (void)hipFree(p);
      return hipErrorOutOfMemory;
    }
    *out = p;
    return hipSuccess;
  } catch (...) {
    return hipErrorOutOfMemory;
  }
}

hipError_t pool_free(void* p, bool idle) {
  try {
    Pool& P = pool();
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.used.find(p);
    if (it == P.used.end()) return hipFree(p);   // not from the pool
    Block b = it->second;
    P.used.erase(it);
    int cur = 0;
    bool keep = idle && hipGetDevice(&cur) == hipSuccess && cur == b.dev;   // (another device's limits are not at hand)
    if (keep) {
      Idle& d = P.idle_of[b.dev];
      d.unseen += b.cap;
      if (d.unseen >= kLookEvery) {
        size_t free_b = 0, total_b = 0;
        keep = hipMemGetInfo(&free_b, &total_b) == hipSuccess;
        d.bound = keep ? std::min(total_b / 8, free_b) : 0;
        d.unseen = keep ? 0 : kLookEvery;
      }
      keep = keep && b.cap <= d.bound;
      trim(P, b.dev, keep ? d.bound - b.cap : d.bound, kMaxIdle - 1);
    }
    if (keep) {
      try {
        Idle& d = P.idle_of[b.dev];
        P.idle.push_back(b);
        d.bytes += b.cap;
        d.count += 1;
        return hipSuccess;
      } catch (...) {
      }
    }
    return hipFree(p);
  } catch (...) {
    return hipErrorOutOfMemory;
  }
}

size_t pool_release() {
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  size_t n = 0;
  for (auto it = P.idle.begin(); it != P.idle.end(); it = drop(P, it)) {
    n += it->cap;
    (void)hipFree(it->p);
  }
  return n;
}

hipError_t mem_available(size_t* free_bytes, size_t* total_bytes) {
  hipError_t e = hipMemGetInfo(free_bytes, total_bytes);
  int dev = 0;
  if (e == hipSuccess) e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  Pool& P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  const auto it = P.idle_of.find(dev);
  if (it != P.idle_of.end()) *free_bytes += it->second.bytes;
  return hipSuccess;
}

}  // namespace kpm

extern "C" int kpm_release_workspace(int64_t* bytes) {
  try {
    kpm::clear_error();
    const size_t n = kpm::pool_release();
    if (bytes) *bytes = (int64_t)n;
    return KPM_OK;
  } catch (...) {
    kpm::set_error("internal error (exception) in kpm_release_workspace");
    return KPM_E_DEVICE;
  }
}
