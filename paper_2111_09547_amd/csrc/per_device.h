// State that belongs to a device and not to the process.
#pragma once
#include <stdint.h>

#include <atomic>

namespace qgtc {

// Something that has to be done once on every device, by whichever thread comes first: set()
// returns whether it worked, and is tried again by the next caller if it did not.  (Two threads
// that come together may both do it.)
class OncePerDevice {
 public:
  template <class Set>
  bool operator()(int dev, Set set) {
    if (dev < 0) return false;
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0u;   // (devices past 64: every time)
    if (done_.load(std::memory_order_acquire) & bit) return true;
    if (!set()) return false;
    done_.fetch_or(bit, std::memory_order_release);
    return true;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace qgtc
