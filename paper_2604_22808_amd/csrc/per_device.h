#pragma once
// Settings that belong to a device's copy of a kernel (its limit of dynamic LDS): made once on every device a process uses.
#include <atomic>
#include <cstdint>

namespace fa {

class OncePerDevice {
  std::atomic<uint64_t> done_{0};

 public:
  // Calls set(), which returns 0 on success, unless it has succeeded for `device` before, and returns its result.  Two threads
  // that meet here may both call it; neither goes on before it has succeeded once.
  template <typename F>
  int run(int device, F&& set) {
    const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;   // (other devices: every time)
    if (bit && (done_.load(std::memory_order_acquire) & bit)) return 0;
    const int e = set();
    if (e == 0) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }
};

}  // namespace fa
