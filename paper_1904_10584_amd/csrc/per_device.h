// Something done once for every device of the process.
#pragma once

#include <stdint.h>

#include <atomic>

namespace am {

// Safe with several threads (two may both do it); a failure is not remembered.
// Device numbers beyond 63 do it every time.
struct PerDevice {
  std::atomic<uint64_t> done{0};
  template <typename F> auto once(int device, F&& f) -> decltype(f()) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    using R = decltype(f());
    if (done.load(std::memory_order_acquire) & bit) return R{};
    const R r = f();
    if (r == R{}) done.fetch_or(bit, std::memory_order_release);
    return r;
  }
};

}  // namespace am
