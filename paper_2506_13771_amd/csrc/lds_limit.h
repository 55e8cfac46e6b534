// A kernel's dynamic LDS limit beyond the default 64 KB, raised per device (the
// attribute belongs to the device current at the call) and only upwards, so that
// calls captured in a graph after an eager call of the same shape make no
// attribute call.  Free of HIP: the caller gives the device and the setter.
#pragma once
#include <atomic>
#include <cstddef>
#include <cstdint>
#include <mutex>

namespace lb {

class LdsLimit {
 public:
  static constexpr size_t kDefault = 65536;
  static constexpr int kDevices = 16;
  // device(int*) and set(size_t) return 0 on success; so does raise
  template <typename Device, typename Set>
  int raise(size_t bytes, Device device, Set set) {
    if (bytes <= kDefault) return 0;
    int dev = 0;
    if (const int e = device(&dev)) return e;
    if (dev < 0 || dev >= kDevices) return set(bytes);
    const uint32_t want = static_cast<uint32_t>(bytes);
    if (want <= limit_[dev].load(std::memory_order_acquire)) return 0;
    std::lock_guard<std::mutex> lock(mu_);
    if (want <= limit_[dev].load(std::memory_order_relaxed)) return 0;
    if (const int e = set(bytes)) return e;
    limit_[dev].store(want, std::memory_order_release);
    return 0;
  }

 private:
  std::atomic<uint32_t> limit_[kDevices] = {};
  std::mutex mu_;
};

}  // namespace lb
