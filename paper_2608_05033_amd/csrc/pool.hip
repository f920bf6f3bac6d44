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
// would have made at once, and only where no idle block of its size is there.
// sd_release_memory, or an allocation that would otherwise fail, returns the
// kept blocks to the device.
//
// The lock covers the lists alone: no HIP call is made under it, so a thread
// that waits for its device holds up neither another device's threads nor its own's.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <mutex>
#include <new>
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
  uint64_t age;
};
struct DevicePool {
  using Blocks = std::multimap<size_t, Kept>;  // by size
  struct Place {
    bool in_flight;
    Blocks::iterator it;
  };
  Blocks idle, in_flight;
  std::map<uint64_t, Place> ages;  // the longest kept first
  size_t kept = 0;
  uint64_t next_age = 0;

  void add(size_t bytes, void *p, bool flying) {  // may throw: nothing is added then
    Blocks &to = flying ? in_flight : idle;
    auto it = to.emplace(bytes, Kept{p, next_age});
    try {
      ages.emplace(next_age, Place{flying, it});
    } catch (...) {
      to.erase(it);
      throw;
    }
    ++next_age;
    kept += bytes;
  }
  void *take(Place at) {
    void *p = at.it->second.p;
    kept -= at.it->first;
    ages.erase(at.it->second.age);
    (at.in_flight ? in_flight : idle).erase(at.it);
    return p;
  }
  // The smallest block of `size` to 5/4 `size` bytes; of two of one size (sizes come in
  // steps of about an eighth) the idle one.  A larger idle block is not taken instead: it is
  // then missing where its size is asked for, and the next matrix's plan maps memory again
  // (R-MAT 143 k vertices, 2.9 M edges, first sd_plan_device + sd_spmm of a second
  // matrix: 450 us, 530 with any idle block that fits first).
  bool find(size_t size, Place *at) {
    auto i = idle.lower_bound(size), f = in_flight.lower_bound(size);
    const size_t most = size + size / 4;
    const bool idle_fits = i != idle.end() && i->first <= most;
    const bool flying_fits = f != in_flight.end() && f->first <= most;
    if (!idle_fits && !flying_fits) return false;
    const bool flying = flying_fits && (!idle_fits || f->first < i->first);
    *at = {flying, flying ? f : i};
    return true;
  }
  // What was kept before `age` is no longer in flight.
  void drained(uint64_t age) {
    for (auto it = in_flight.begin(); it != in_flight.end();) {
      auto here = it++;
      if (here->second.age >= age) continue;
      const uint64_t a = here->second.age;
      ages[a] = {false, idle.insert(in_flight.extract(here))};
    }
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

// 4 KiB steps up to 64 KiB, then eighths of the next power of two below.  What is too
// large to be kept is not stretched.
size_t rounded(size_t bytes) {
  size_t step = 4096;
  while (step * 16 < bytes && bytes <= kKeep) step *= 2;
  return (bytes + step - 1) / step * step;
}

// Frees the kept blocks of a device; hipFree waits.
void release_kept(Pool &P, int device) {
  for (;;) {
    void *p = nullptr;
    {
      std::lock_guard<std::mutex> lock(P.mu);
      DevicePool &D = P.dev.at(device);
      if (D.ages.empty()) return;
      p = D.take(D.ages.begin()->second);
    }
    (void)hipFree(p);
  }
}

// A kept block that fits, nothing pending on it; null if there is none.
void *take_kept(Pool &P, int dev, size_t size) {
  void *p = nullptr;
  uint64_t before = 0;
  {
    std::lock_guard<std::mutex> lock(P.mu);
    DevicePool &D = P.dev[dev];
    DevicePool::Place at;
    if (!D.find(size, &at)) return nullptr;
    P.live.emplace(at.it->second.p, Block{dev, at.it->first});  // may throw: before the block leaves the list
    p = D.take(at);
    if (!at.in_flight) return p;
    before = D.next_age;
  }
  if (hipDeviceSynchronize() != hipSuccess) {  // a capture is under way, say: not this one
    (void)hipGetLastError();
    pool_free(p, kInFlight);
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(P.mu);
  P.dev.at(dev).drained(before);
  return p;
}

}  // namespace

hipError_t pool_alloc(void **out, size_t bytes) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (!bytes) bytes = 1;
  size_t size = rounded(bytes);
  Pool &P = pool();
  try {
    if ((*out = take_kept(P, dev, size))) return hipSuccess;
    void *q = nullptr;
    e = hipMalloc(&q, size);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      release_kept(P, dev);
      e = hipMalloc(&q, size);
    }
    if (e == hipErrorOutOfMemory && size > bytes) {
      (void)hipGetLastError();
      e = hipMalloc(&q, size = bytes);
    }
    if (e != hipSuccess) return e;
    try {
      std::lock_guard<std::mutex> lock(P.mu);
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
  Block b;
  {
    std::lock_guard<std::mutex> lock(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) return;
    b = it->second;
    P.live.erase(it);
  }
  while (state != kUnknown && b.bytes <= kKeep) {
    void *oldest = nullptr;
    {
      std::lock_guard<std::mutex> lock(P.mu);
      DevicePool &D = P.dev.at(b.device);
      if (D.kept + b.bytes <= kKeep) {
        try {
          D.add(b.bytes, p, state == kInFlight);
          return;
        } catch (const std::bad_alloc &) {
          break;
        }
      }
      oldest = D.take(D.ages.begin()->second);
    }
    (void)hipFree(oldest);
  }
  (void)hipFree(p);
}

}  // namespace sd

extern "C" void sd_release_memory(void) {
  sd::Pool &P = sd::pool();
  for (int device = -1;;) {
    {
      std::lock_guard<std::mutex> lock(P.mu);
      auto next = P.dev.upper_bound(device);
      if (next == P.dev.end()) return;
      device = next->first;
    }
    sd::release_kept(P, device);
  }
}
