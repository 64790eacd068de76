// Settings of a kernel that hold for one device.
#pragma once
#include <atomic>
#include <cstdint>

namespace betty {

// Runs a setting once for every device, from any thread (two first calls on a device may both run it, which does no
// harm to a setting).  One that fails is tried again at the next call; devices from 64 on run it every time.
class PerDevice {
  std::atomic<uint64_t> done{0};
 public:
  template <typename F> bool once(int device, F set) {
    const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return true;
    if (!set()) return false;
    if (bit) done.fetch_or(bit, std::memory_order_release);
    return true;
  }
};

}  // namespace betty
