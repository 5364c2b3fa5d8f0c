// Something that is done once for every device.
#ifndef SPTIR_PER_DEVICE_H_
#define SPTIR_PER_DEVICE_H_

#include <atomic>
#include <cstdint>

namespace sptir {

// do_it() returns whether it succeeded, and may be repeated: threads that come at the same time all do it, so that none goes on
// before it is done.  Devices beyond the first 64 have it done every time.
class OncePerDevice {
 public:
  template <typename F>
  void operator()(int device, F&& do_it) {
    const bool kept = device >= 0 && device < 64;
    const uint64_t bit = kept ? (uint64_t)1 << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return;
    if (do_it()) done_.fetch_or(bit, std::memory_order_release);
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace sptir

#endif  // SPTIR_PER_DEVICE_H_
