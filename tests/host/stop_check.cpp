// Host-side check of a workgroup's decision on a word that others write
// meanwhile (no GPU, no HIP): compiled with g++ by tests/test_host_stop.py.
#include <stdio.h>

#include <atomic>
#include <condition_variable>
#include <mutex>
#include <thread>
#include <vector>

#include "build_plan.hpp"

using namespace compass;

// Waves of one workgroup as threads; `bad` turns 1 after `after` loads of it.
constexpr int kWaves = 16;

struct Barrier {
  std::mutex mu;
  std::condition_variable cv;
  int waiting = 0, phase = 0;
  void operator()() {
    std::unique_lock<std::mutex> lk(mu);
    const int p = phase;
    if (++waiting == kWaves) {
      waiting = 0;
      ++phase;
      cv.notify_all();
    } else {
      cv.wait(lk, [&] { return phase != p; });
    }
  }
};

int main() {
  int fails = 0;
  for (int after = 0; after <= kWaves; ++after) {
    std::atomic<int> loads{0};
    Barrier barrier;
    uint32_t word = 7;
    std::atomic<int> leave{0};
    std::vector<std::thread> waves;
    for (int w = 0; w < kWaves; ++w)
      waves.emplace_back([&, w] {
        if (block_reads(&word, w == 0, [&] { return loads++ >= after ? 1u : 0u; },
                        [&] { barrier(); }))
          ++leave;
      });
    for (auto &t : waves) t.join();
    if (leave != 0 && leave != kWaves) {
      printf("FAIL: %d of %d waves leave (flag raised at load %d)\n", leave.load(), kWaves,
             after);
      ++fails;
    }
    if (loads != 1) {
      printf("FAIL: the word was loaded %d times\n", loads.load());
      ++fails;
    }
  }
  if (!fails) printf("ok\n");
  return fails != 0;
}
