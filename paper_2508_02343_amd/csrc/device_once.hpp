// Something done once on each device, from any thread.  No HIP: tests compile
// it by itself.
#pragma once

#include <stdint.h>

#include <atomic>

namespace mm {

class DeviceOnce {
 public:
  // Runs f unless it has succeeded (returned 0) on this device before, and gives
  // its result.  Threads that come at the same time may each run it.
  template <typename F>
  int run(int device, F f) {
    const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;  // (others: every time)
    if (done_.load(std::memory_order_acquire) & bit) return 0;
    const int e = f();
    if (e == 0) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace mm
