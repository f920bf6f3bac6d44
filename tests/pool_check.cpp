// The device memory pool against a fake HIP of two devices with 16 GiB each.
// Usage: pool_check CASE; exit status 0 if the case holds.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

#include "kernels.h"

extern "C" void sd_release_memory(void);

namespace {
std::mutex mu;
std::map<uintptr_t, std::pair<int, size_t>> blocks;  // address -> device, bytes
size_t used[2];
uintptr_t next_address = 1 << 20;
std::atomic<int> syncs{0}, mallocs{0};
std::atomic<bool> hold_sync{false}, in_sync{false};
thread_local int device = 0;
constexpr size_t kMemory = (size_t)16 << 30, GiB = (size_t)1 << 30, MiB = (size_t)1 << 20;
}  // namespace

hipError_t hipMalloc(void **p, size_t bytes) {
  std::lock_guard<std::mutex> lock(mu);
  ++mallocs;
  if (used[device] + bytes > kMemory) return hipErrorOutOfMemory;
  used[device] += bytes;
  blocks[next_address] = {device, bytes};
  *p = reinterpret_cast<void *>(next_address);
  next_address += bytes + 4096;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  std::lock_guard<std::mutex> lock(mu);
  auto it = blocks.find(reinterpret_cast<uintptr_t>(p));
  if (it == blocks.end()) return hipErrorUnknown;
  used[it->second.first] -= it->second.second;
  blocks.erase(it);
  return hipSuccess;
}
hipError_t hipGetDevice(int *dev) {
  *dev = device;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  ++syncs;
  in_sync = true;
  while (hold_sync) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  in_sync = false;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }

#define CHECK(x)                                                 \
  do {                                                           \
    if (!(x)) {                                                  \
      std::printf("line %d: %s\n", __LINE__, #x);                \
      std::fflush(stdout);                                       \
      std::_Exit(1);                                             \
    }                                                            \
  } while (0)

static void *take(size_t bytes, hipError_t want = hipSuccess) {
  void *p = nullptr;
  const hipError_t e = sd::pool_alloc(&p, bytes);
  CHECK(e == want);
  return p;
}

// While one device's work is waited for, the other device allocates and frees.
static void devices_apart() {
  void *a = take(MiB);
  sd::pool_free(a, sd::kInFlight);
  hold_sync = true;
  std::thread first([&] {
    device = 0;
    sd::pool_free(take(MiB), sd::kIdle);  // takes the block in flight: waits for device 0
  });
  while (!in_sync) std::this_thread::yield();
  std::atomic<bool> done{false};
  std::thread second([&] {
    device = 1;
    void *b = take(2 * MiB);
    sd::pool_free(b, sd::kIdle);
    CHECK(take(2 * MiB) == b);
    done = true;
  });
  for (int t = 0; t < 2000 && !done; ++t) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  const bool apart = done;
  hold_sync = false;
  first.join();
  second.join();
  CHECK(apart);
}

// An idle block is taken before one of its size that has to be waited for; a larger idle
// one is kept for requests of its own size.
static void idle_first() {
  void *busy = take(MiB), *idle = take(MiB - 100), *large = take(MiB + MiB / 8);
  sd::pool_free(busy, sd::kInFlight);
  sd::pool_free(idle, sd::kIdle);
  sd::pool_free(large, sd::kIdle);
  CHECK(take(MiB - 10) == idle && syncs == 0);
  CHECK(take(MiB) == busy && syncs == 1);  // nothing else of its size is left
  CHECK(take(MiB) == large && syncs == 1 && mallocs == 3);
  // blocks given back while a synchronisation runs are not covered by it
  sd::pool_free(busy, sd::kInFlight);
  hold_sync = true;
  std::thread other([&] { sd::pool_free(take(MiB), sd::kIdle); });
  while (!in_sync) std::this_thread::yield();
  sd::pool_free(idle, sd::kInFlight);
  hold_sync = false;
  other.join();
  CHECK(syncs == 2);
  CHECK(take(MiB) == busy && syncs == 2);  // idle again
  CHECK(take(MiB) == idle && syncs == 3);  // still in flight
}

// What the device can hold is given out: no rounding stands in the way, kept blocks do not.
static void all_memory() {
  void *a = take(15 * GiB + 3);  // 15/16 of the device: no step of it is added
  CHECK(used[0] <= 15 * GiB + 4096);
  void *b = take(GiB - 8 * MiB);  // rounded it would not fit any more
  sd::pool_free(b, sd::kIdle);
  CHECK(take(GiB - 4 * MiB) != nullptr);  // the kept block makes room
  take(64 * MiB, hipErrorOutOfMemory);
  sd::pool_free(a, sd::kInFlight);  // too large to keep
  CHECK(used[0] < GiB + MiB);
}

// At most 1 GiB is kept per device, the newest; all of it can be given back.
static void bounded() {
  void *p[40];
  for (auto &q : p) q = take(64 * MiB);
  for (auto &q : p) sd::pool_free(q, sd::kIdle);
  CHECK(used[0] == GiB);
  CHECK(take(64 * MiB) != p[0]);
  device = 1;
  sd::pool_free(take(MiB), sd::kIdle);
  CHECK(used[1] == MiB);
  sd_release_memory();
  CHECK(used[0] == 64 * MiB && used[1] == 0);
  sd::pool_free(take(MiB), sd::kUnknown);
  CHECK(used[1] == 0);
}

// Threads on both devices: no block is in two hands, all of it comes back.
static void threads() {
  std::mutex owned_mu;
  std::map<void *, int> owned;
  std::thread t[8];
  for (int i = 0; i < 8; ++i)
    t[i] = std::thread([&, i] {
      device = i & 1;
      uint32_t x = 12345u + (uint32_t)i;
      for (int turn = 0; turn < 3000; ++turn) {
        void *q[3];
        for (auto &p : q) {
          x = x * 1664525u + 1013904223u;
          p = take(4096 + (x >> 8) % (8 * MiB));
          std::lock_guard<std::mutex> lock(owned_mu);
          CHECK(owned.emplace(p, i).second);
        }
        for (auto &p : q) {
          x = x * 1664525u + 1013904223u;
          {
            std::lock_guard<std::mutex> lock(owned_mu);
            owned.erase(p);
          }
          sd::pool_free(p, x >> 31 ? sd::kIdle : sd::kInFlight);
        }
        if (turn % 500 == 499) sd_release_memory();
      }
    });
  for (auto &x : t) x.join();
  sd_release_memory();
  CHECK(used[0] == 0 && used[1] == 0);
}

int main(int argc, char **argv) {
  const char *name = argc > 1 ? argv[1] : "";
  struct {
    const char *name;
    void (*run)();
  } cases[] = {{"devices_apart", devices_apart}, {"idle_first", idle_first}, {"all_memory", all_memory},
               {"bounded", bounded}, {"threads", threads}};
  for (auto &c : cases)
    if (!std::strcmp(c.name, name)) {
      c.run();
      return 0;
    }
  return 2;
}
