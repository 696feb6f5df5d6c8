// Host check of LdsLimit (csrc/qpg_internal.hpp) with several threads: after raise(bytes) the attribute is at least
// `bytes`, whatever other threads raise it to. The attribute is a variable per device, written after a pause.
#include <chrono>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "qpg_internal.hpp"

int main() {
  for (int device : {0, 63, 64, -1}) {
    for (int round = 0; round < 40; ++round) {
      qpg::LdsLimit limit;
      std::atomic<size_t> attribute{0};
      std::atomic<int> wrong{0}, sets{0};
      std::vector<std::thread> th;
      for (int t = 0; t < 4; ++t)
        th.emplace_back([&, t] {
          std::mt19937 rng((unsigned)(40 * t + round));
          for (int k = 0; k < 8; ++k) {
            const size_t bytes = rng() % 160 * 1024;
            limit.raise(device, bytes, [&](size_t most) {
              ++sets;
              std::this_thread::sleep_for(std::chrono::microseconds(rng() % 50));
              attribute = most;
            });
            if (attribute < bytes) ++wrong;
          }
        });
      for (auto& x : th) x.join();
      if (wrong || (device >= 0 && device < 64 && sets > 32)) {
        std::printf("device %d: %d launches above the limit, %d sets\n", device, wrong.load(), sets.load());
        return 1;
      }
    }
  }
  return 0;
}
