// Sizes of the far-field expansions (dpr1_kernels.hip): how many records a
// problem has and how many blocks form them.  Host arithmetic only.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace dpr1 {

constexpr int WAVE = 64;
constexpr int FAR_WIDE = 8;  // blocks of 64 eigenvalues that share a wide record
constexpr int FAR_SLICE = 2048, FAR_NSL_MAX = 1024;

// Orders from which a problem has records, and from which it has the wide
// level too.  Below FAR_MIN the near window of a block (about 2.5 times its
// 64 poles) is most of the problem.
constexpr int FAR_MIN = 384, FAR_MIN2 = 2048;
static constexpr int64_t far_slices(int64_t n) {
  const int64_t s = (n + FAR_SLICE - 1) / FAR_SLICE;
  return s > FAR_NSL_MAX ? FAR_NSL_MAX : s;
}
// records of the wide level
static constexpr int64_t far_wide_records(int64_t n) {
  if (n < FAR_MIN2) return 0;
  return ((n + WAVE - 1) / WAVE + FAR_WIDE - 1) / FAR_WIDE * far_slices(n);
}

// Blocks of k_far (FAR_BLK threads each), which loop over the records: one a
// record up to FAR_GRID, far more than the GPU holds and far below the 2^32
// threads that a launch may have.
constexpr int FAR_BLK = 256;
constexpr int64_t FAR_GRID = 1 << 20;
static constexpr int64_t far_grid(int64_t records) { return records < FAR_GRID ? records : FAR_GRID; }

}  // namespace dpr1
