// A per-kernel setting that belongs to a device (the dynamic LDS a launch may ask for): made once for
// each device that launches the kernel, from whatever thread.
#pragma once
#include <atomic>
#include <cstdint>

namespace bs {

class OncePerDevice {
  std::atomic<uint64_t> made_{0};  // one bit per device

 public:
  // Runs `make` (0 = success) unless it has succeeded for `device`; what fails, and devices beyond 63, run again.
  // Two threads may run it at the same time: the setting is the same.
  template <class Make>
  int operator()(int device, Make &&make) {
    const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;
    if (made_.load(std::memory_order_acquire) & bit) return 0;
    const int rc = make();
    if (rc == 0) made_.fetch_or(bit, std::memory_order_release);
    return rc;
  }
};

}  // namespace bs
