// Flat indices over the threads of a launch.  Plain C++, so that the host can check them too.
#pragma once

#include <stdint.h>

namespace kvc {

// 64 bits throughout: 65535 (layer, head) pairs x 256 sequences x 1024 threads, which every limit
// of a call allows, are 2^34 threads.
constexpr int64_t flat_thread(uint32_t bx, uint32_t by, uint32_t gx, uint32_t threads, uint32_t thread) {
  return (int64_t(by) * gx + bx) * threads + thread;
}
constexpr int64_t grid_threads(uint32_t gx, uint32_t gy, uint32_t threads) {
  return int64_t(gx) * gy * threads;
}

}  // namespace kvc
