// spin_once.h -- calls made once per device, from any thread (a kernel's LDS limit is set for a function on
// a device).
#pragma once

#include <stdint.h>

#include <atomic>

namespace spin {

class OncePerDevice {
 public:
  // ok where the call has succeeded on this device before, else its result.  Threads that meet here may
  // each make it.
  template <class R, class F>
  R run(int device, R ok, F call) {
    const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;  // further devices: every time
    if (done_.load(std::memory_order_acquire) & bit) return ok;
    const R r = call();
    if (r == ok) done_.fetch_or(bit, std::memory_order_release);
    return r;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace spin
