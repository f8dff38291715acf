// Host bookkeeping of what has to be done once on every GPU that the process uses.
#pragma once
#include <atomic>
#include <cstdint>

namespace esa {

// done(dev) turns true for a device once mark(dev) was called for that device (device numbers from 64 on: never, the work
// is then repeated).  Threads may find it false together and repeat the work, which must allow for that.
class OncePerDevice {
 public:
  bool done(int dev) const { return dev >= 0 && dev < 64 && ((bits_.load(std::memory_order_acquire) >> dev) & 1u); }
  void mark(int dev) {
    if (dev >= 0 && dev < 64) bits_.fetch_or((uint64_t)1 << dev, std::memory_order_release);
  }

 private:
  std::atomic<uint64_t> bits_{0};
};

}  // namespace esa
