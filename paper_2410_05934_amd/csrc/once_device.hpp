// once_device.hpp -- a setting made once per device, from any thread.
#pragma once

#include <atomic>
#include <cstdint>

namespace nttk {

// run(device, f) calls f() until it has returned 0 once for that device and returns
// what it returned (0 ever after).  Threads that come first together may each call it,
// so f sets the same value every time.  Devices past 63 set it on every call.
class OncePerDevice {
 public:
  template <class F>
  auto run(int device, F f) -> decltype(f()) {
    const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return decltype(f())(0);
    const auto e = f();
    if (e == decltype(f())(0)) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace nttk
