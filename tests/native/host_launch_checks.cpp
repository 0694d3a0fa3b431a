// The launchers' host helpers, without a GPU.  OncePerDevice (which devices a kernel's attribute was set on): every device
// gets its own call, a failure is not remembered, and many host threads may come at once (run under ThreadSanitizer).
// launch_grid: fewer than 2^32 threads per dimension, no workgroup left out, whole multiples of the eight XCDs per row.
#include <cstdio>
#include <thread>
#include <vector>

#include "../../paper_2508_02322_amd/csrc/host_launch.h"

static std::atomic<int> failures{0};
#define EXPECT(cond)                                                                \
  do {                                                                              \
    if (!(cond)) {                                                                  \
      std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
      ++failures;                                                                   \
    }                                                                               \
  } while (0)

int main() {
  camera::OncePerDevice once;
  int calls = 0;
  auto good = [&] { ++calls; return hipSuccess; };
  auto bad = [&] { ++calls; return hipErrorInvalidValue; };
  EXPECT(once(0, bad) == hipErrorInvalidValue && calls == 1);
  EXPECT(once(0, good) == hipSuccess && calls == 2);   // the failure was not remembered
  EXPECT(once(0, bad) == hipSuccess && calls == 2);    // the success is
  for (int device = 1; device < 64; ++device) EXPECT(once(device, good) == hipSuccess && calls == 2 + device);
  for (int device = 0; device < 64; ++device) EXPECT(once(device, bad) == hipSuccess);
  EXPECT(calls == 65);
  EXPECT(once(64, good) == hipSuccess && once(64, good) == hipSuccess && calls == 67);

  camera::OncePerDevice shared;
  std::atomic<int> per_device[8] = {};
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      for (int i = 0; i < 1000; ++i) {
        const int device = (t + i) % 8;
        EXPECT(shared(device, [&] { ++per_device[device]; return hipSuccess; }) == hipSuccess);
      }
    });
  for (auto& t : threads) t.join();
  for (auto& n : per_device) EXPECT(n >= 1 && n <= 8);  // threads that come together may each set it
  for (int64_t blocks : {int64_t(1), int64_t(255), (int64_t(1) << 22) - 1, int64_t(1) << 22, (int64_t(1) << 22) + 1, int64_t(1) << 24,
                         (int64_t(1) << 28) + 5, (int64_t(1) << 31) - 1}) {
    const dim3 g = camera::launch_grid(blocks);
    EXPECT((uint64_t)g.x * 512 < (uint64_t(1) << 32) && g.y >= 1 && g.z == 1);
    EXPECT((int64_t)g.x * g.y >= blocks && (g.y == 1 || (g.x == (1u << camera::kGridWidthLog2) && g.x % 8 == 0)));
    EXPECT((int64_t)g.x * (g.y - 1) < blocks);
  }

  if (!failures) std::printf("host launch: all passed\n");
  return failures ? 1 : 0;
}
