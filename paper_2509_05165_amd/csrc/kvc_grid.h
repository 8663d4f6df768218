// Index arithmetic over the grid of a launch.  Plain C++, so that the host can check it too.
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

// Order of the workgroups of a score launch whose last row chunk is short.  A launch has
// slices = gx * hkv * gz stretches of K, each worked by row_chunks workgroups: row_chunks - 1 long
// ones and a short one.  They go out in groups of GRID_GROUP slices: the first row chunks of all
// slices of a group, then the second ones, and so on.  Workgroup p of the launch stands for block
// (bx, by, bz) of the grid (gx, hkv * row_chunks, gz), and p = 0 for (0, 0, 0).
//
// 256 is the number of compute units.  Consecutive workgroups go to consecutive XCDs, shader engines
// and compute units, and a compute unit holds two: a group puts one long workgroup on every unit
// and one short one beside it, the row chunks of a slice meet on one XCD (256 is a multiple of 8),
// and the K of a group, 134 or 268 MB at most, is mostly still in the memory-side cache when the
// short ones ask for it.
constexpr uint32_t GRID_GROUP = 256;
struct GridBlock { uint32_t bx, by, bz; };
constexpr GridBlock row_chunk_block(uint32_t p, uint32_t gx, uint32_t hkv, uint32_t row_chunks, uint32_t gz) {
  const uint32_t slices = gx * hkv * gz;
  const uint32_t first = p / (GRID_GROUP * row_chunks) * GRID_GROUP;      // of the group
  const uint32_t left = slices - first, here = left < GRID_GROUP ? left : GRID_GROUP;
  const uint32_t q = p - first * row_chunks, rc = q / here;
  const uint32_t slice = first + q - rc * here;
  const uint32_t lh = slice / gx, bz = lh / hkv;
  return {slice - lh * gx, (lh - bz * hkv) * row_chunks + rc, bz};
}

// The same for batches of unequal sequences: the stretches of K of a sequence's (layer, head) pairs together,
// bx slowest, so that what bx counts last (the short ones) is worked last and the workgroups that
// are still running when no others are left are short.
constexpr GridBlock pair_major_block(uint32_t p, uint32_t gx, uint32_t hkv, uint32_t row_chunks, uint32_t gz) {
  const uint32_t slices = gx * hkv * gz;
  const uint32_t first = p / (GRID_GROUP * row_chunks) * GRID_GROUP;      // of the group
  const uint32_t left = slices - first, here = left < GRID_GROUP ? left : GRID_GROUP;
  const uint32_t q = p - first * row_chunks, rc = q / here;
  const uint32_t slice = first + q - rc * here;
  const uint32_t bx = slice / (hkv * gz), lh = slice - bx * (hkv * gz), bz = lh / hkv;
  return {bx, (lh - bz * hkv) * row_chunks + rc, bz};
}

}  // namespace kvc
