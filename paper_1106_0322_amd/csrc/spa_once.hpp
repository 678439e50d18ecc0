// Bookkeeping of what is done once per device: a kernel's limit of dynamic LDS is an attribute of
// its copy on one device, so a process-wide flag leaves the kernel refused on the second device.
#pragma once

#include <atomic>
#include <cstdint>

namespace spa {

// Whether `act(device)` has succeeded (returned true) for a device; safe with several threads
// (two that come first together both act).  Devices beyond 63 act every time.
class OncePerDevice {
 public:
  template <typename Act>
  bool run(int device, Act act) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return true;
    if (!act(device)) return false;
    done_.fetch_or(bit, std::memory_order_release);
    return true;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace spa
