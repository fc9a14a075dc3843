// Set-up that is needed once per device of the process.
#pragma once
#include <atomic>
#include <cstdint>

namespace cf {

// run(device, set_up) calls set_up unless a call of it for that device has ended before.  Threads that
// arrive together may each call it (it has to bear that); none goes on before a call for its device has
// ended.  Devices from 64 on are set up every time.
class PerDevice {
  public:
    template <typename F> void run(int device, F&& set_up) {
        const uint64_t bit = device >= 0 && device < 64 ? (uint64_t)1 << device : 0;
        if (done_.load(std::memory_order_acquire) & bit) return;
        set_up();
        done_.fetch_or(bit, std::memory_order_release);
    }

  private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace cf
