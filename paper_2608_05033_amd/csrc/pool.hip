// Device memory for plans and conversion scratch, kept for reuse.
//
// Mapping and unmapping device memory is what a plan build waits on once its
// kernels are short: above a few MB one hipMalloc or hipFree took 20-450 us
// here, and a plan with its scratch makes about 20 of them (R-MAT 500 k
// vertices, 8 M edges: 1.7 of the 3.6 ms of sd_plan_device + sd_spmm +
// sd_plan_destroy).  Freed blocks are kept per device up to kKeep bytes, the
// longest kept making room, and handed out again, best fit within a quarter of
// the size asked for.
//
// A block may be handed to any stream, so nothing that uses it may be pending by
// then: scratch is given back after its stream has drained (kIdle); a plan's
// memory may still be read by products its caller has in flight (kInFlight),
// and is handed out again only after a device synchronisation, which hipFree
// would have made at once.  sd_release_memory, or an allocation that would
// otherwise fail, returns the kept blocks to the device.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <mutex>
#include <unordered_map>

#include "kernels.h"

namespace sd {
namespace {

constexpr size_t kKeep = (size_t)1 << 30;  // bytes kept per device (288 GB each)

struct Block {
  int device;
  size_t bytes;
};
struct Kept {
  void *p;
  bool in_flight;
  uint64_t age;
};
struct DevicePool {
  std::multimap<size_t, Kept> blocks;                              // by size
  std::map<uint64_t, std::multimap<size_t, Kept>::iterator> ages;  // the longest kept first
  size_t kept = 0;
  uint64_t next_age = 0;

  void add(size_t bytes, void *p, bool in_flight) {  // may throw: nothing is added then
    auto it = blocks.emplace(bytes, Kept{p, in_flight, next_age});
    try {
      ages.emplace(next_age, it);
    } catch (...) {
      blocks.erase(it);
      throw;
    }
    ++next_age;
    kept += bytes;
  }
  void *take(std::multimap<size_t, Kept>::iterator it) {
    void *p = it->second.p;
    kept -= it->first;
    ages.erase(it->second.age);
    blocks.erase(it);
    return p;
  }
};
struct Pool {
  std::mutex mu;
  std::unordered_map<void *, Block> live;
  std::map<int, DevicePool> dev;
};
// Never destroyed: plans may be freed while the process ends.
Pool &pool() {
  static Pool *p = new Pool;
  return *p;
}

// 4 KiB steps up to 64 KiB, then eighths of the next power of two below.
size_t rounded(size_t bytes) {
  size_t step = 4096;
  while (step * 16 < bytes) step *= 2;
  return (bytes + step - 1) / step * step;
}

// Frees every kept block of a device (-1: of all devices); hipFree waits.
void release_kept(Pool &P, int device) {
  for (auto &d : P.dev) {
    if (device >= 0 && d.first != device) continue;
    while (!d.second.blocks.empty()) (void)hipFree(d.second.take(d.second.blocks.begin()));
  }
}

}  // namespace

hipError_t pool_alloc(void **out, size_t bytes) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const size_t size = rounded(bytes ? bytes : 1);
  Pool &P = pool();
  try {
    std::lock_guard<std::mutex> lock(P.mu);
    DevicePool &D = P.dev[dev];
    auto it = D.blocks.lower_bound(size);
    bool fits = it != D.blocks.end() && it->first <= size + size / 4;
    if (fits && it->second.in_flight) {
      if (hipDeviceSynchronize() == hipSuccess) {
        for (auto &b : D.blocks) b.second.in_flight = false;
      } else {
        (void)hipGetLastError();
        fits = false;
      }
    }
    if (fits) {
      P.live.emplace(it->second.p, Block{dev, it->first});  // may throw: before the block leaves the list
      *out = D.take(it);
      return hipSuccess;
    }
    void *q = nullptr;
    e = hipMalloc(&q, size);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      release_kept(P, dev);
      e = hipMalloc(&q, size);
    }
    if (e != hipSuccess) return e;
    try {
      P.live.emplace(q, Block{dev, size});
    } catch (...) {
      (void)hipFree(q);
      throw;
    }
    *out = q;
    return hipSuccess;
  } catch (const std::bad_alloc &) {
    return hipErrorOutOfMemory;
  }
}

void pool_free(void *p, PoolState state) {
  if (!p) return;
  Pool &P = pool();
  std::lock_guard<std::mutex> lock(P.mu);
  auto it = P.live.find(p);
  if (it == P.live.end()) return;
  const Block b = it->second;
  P.live.erase(it);
  DevicePool &D = P.dev[b.device];
  if (state != kUnknown && b.bytes <= kKeep) {
    while (D.kept + b.bytes > kKeep) (void)hipFree(D.take(D.ages.begin()->second));
    try {
      D.add(b.bytes, p, state == kInFlight);
      return;
    } catch (const std::bad_alloc &) {
    }
  }
  (void)hipFree(p);
}

}  // namespace sd

extern "C" void sd_release_memory(void) {
  sd::Pool &P = sd::pool();
  std::lock_guard<std::mutex> lock(P.mu);
  sd::release_kept(P, -1);
}
