// Something that has to be done once on every device of the process, by whichever thread gets there first.
#pragma once
#include <atomic>
#include <stdint.h>

namespace dds {

class DeviceOnce {
  std::atomic<uint64_t> done_{0};

 public:
  // True if `act` has succeeded on this device, now or before. Threads that arrive together may all run it; one that
  // fails is run again by the next call. (Devices from 64 on have no bit of their own: they run it every time.)
  template <class Act>
  bool operator()(int device, Act act) {
    if (device < 0 || device >= 64) return act();
    const uint64_t bit = 1ull << device;
    if (done_.load(std::memory_order_acquire) & bit) return true;
    if (!act()) return false;
    done_.fetch_or(bit, std::memory_order_release);
    return true;
  }
};

}  // namespace dds
