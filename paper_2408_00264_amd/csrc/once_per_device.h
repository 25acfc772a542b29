// Host-side set-up that belongs to a GPU and not to the process (the LDS limit of a kernel): done before the first launch
// on every device, from any thread.  Threads that arrive together may both do it; none goes on before it is done.
#pragma once
#include <atomic>
#include <cstdint>

namespace clv {

class OncePerDevice {
 public:
  template <class F>
  void operator()(int device, F&& set_up) {
    if (device < 0 || device >= 64) { set_up(); return; }   // (no bit for it: every time)
    const uint64_t bit = 1ull << device;
    if (done_.load(std::memory_order_acquire) & bit) return;
    set_up();
    done_.fetch_or(bit, std::memory_order_release);
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace clv
