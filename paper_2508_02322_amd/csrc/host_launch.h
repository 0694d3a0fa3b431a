// Host-side helpers of the launchers; no device code, so that a plain C++ program can include them.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace camera {

// A grid of at least `blocks` (< 2^31) workgroups of at most 512 threads, numbered by linear_block().  A launch takes fewer
// than 2^32 threads per dimension, so beyond 2^22 workgroups the numbering goes on in y; the last row may be longer than
// needed.  2^22 is a multiple of the number of XCDs, so consecutive numbers go round them as in a one-dimensional grid.  The
// width is a constant, so that nothing has to be loaded before a workgroup knows its tile.
constexpr int kGridWidthLog2 = 22;
inline dim3 launch_grid(int64_t blocks) {
  constexpr int64_t kWidth = int64_t(1) << kGridWidthLog2;
  return blocks <= kWidth ? dim3((unsigned)blocks) : dim3((unsigned)kWidth, (unsigned)((blocks + kWidth - 1) / kWidth));
}

// A setting that belongs to a device (a kernel's function attribute): set(), which must be repeatable, is called until it
// has succeeded once for that device.  Any host thread, any device; devices beyond the 64 bits are set on every call.
class OncePerDevice {
 public:
  template <class F>
  hipError_t operator()(int device, F&& set) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
    const hipError_t err = set();
    if (err == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
    return err;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace camera
