// A value of each device, asked for once (host code).
#pragma once
#include <atomic>

namespace hfe {
// Threads that ask for a device's value at once may each query it; they store the same.
class PerDevice {
 public:
  // query(dev): the value, positive, or 0 where it cannot be had (not kept)
  template <class F>
  int get(int dev, F query) {
    if (dev < 0 || dev >= kDevices) return query(dev);
    int v = v_[dev].load(std::memory_order_relaxed);
    if (v == 0) {
      v = query(dev);
      v_[dev].store(v, std::memory_order_relaxed);
    }
    return v;
  }

 private:
  static constexpr int kDevices = 64;
  std::atomic<int> v_[kDevices] = {};
};
}  // namespace hfe
