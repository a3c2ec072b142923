// Sizes of the far-field expansions (dpr1_kernels.hip): how many records a
// problem has and how many blocks form them.  Host arithmetic only.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace dpr1 {

constexpr int WAVE = 64;
constexpr int FAR_WIDE = 8;  // blocks of 64 eigenvalues that share a wide record
constexpr int FAR_SLICE = 2048;  // poles of a slice of the wide level, at least

// Orders from which a problem has records, and from which it has the wide
// level too.  Below FAR_MIN the near window of a block (about 2.5 times its
// 64 poles) is most of the problem.
constexpr int FAR_MIN = 384, FAR_MIN2 = 2048;
// Groups of eigenvalues that share a wide expansion, and the slices of the
// poles that each group's moments are formed in, a record a (group, slice).
// Slices are there to fill the GPU: 2048 poles each, but no more than make
// FAR_FILL records in all, or 8 a group where the groups alone are many.  With
// a slice per 2048 poles whatever the order the records were n^2/2^20 (n = 10^6:
// 795 bytes of workspace a row for them); so they are at most 8 a group above
// n = 65536, 13 bytes a row.
constexpr int64_t FAR_FILL = 1024;
static constexpr int64_t far_groups(int64_t n) {
  return ((n + WAVE - 1) / WAVE + FAR_WIDE - 1) / FAR_WIDE;
}
static constexpr int64_t far_slices(int64_t n) {
  const int64_t s = (n + FAR_SLICE - 1) / FAR_SLICE;
  return std::min<int64_t>(s, std::max<int64_t>(FAR_WIDE, FAR_FILL / far_groups(n)));
}
// records of the wide level
static constexpr int64_t far_wide_records(int64_t n) { return n < FAR_MIN2 ? 0 : far_groups(n) * far_slices(n); }
// room for them in a workspace, which may not shrink as n grows (a caller may
// solve smaller problems in the workspace of its largest)
static constexpr int64_t far_wide_room(int64_t n) {
  if (n < FAR_MIN2) return 0;
  return std::min<int64_t>(far_groups(n) * ((n + FAR_SLICE - 1) / FAR_SLICE),
                           std::max<int64_t>(FAR_FILL, FAR_WIDE * far_groups(n)));
}

// Room for the records of a batch of order sum N, largest order nmax and
// `items` blocks of 64 eigenvalues, from what a plan holds, so that a solve can
// check its workspace.  Own records: a problem of order np >= FAR_MIN has
// ceil(np/64) <= np/64 + 63/64 <= 7 np/384 of them.  Wide level: one of order np
// >= FAR_MIN2 has ceil(np/512) <= np/512 + 511/512 <= 5 np/2048 groups.
static constexpr int64_t far_batch_own(int64_t N, int64_t nmax, int64_t items) {
  return nmax < FAR_MIN ? 0 : std::min<int64_t>(items, 7 * N / 384);
}
static constexpr int64_t far_batch_wide(int64_t N, int64_t nmax) {
  if (nmax < FAR_MIN2) return 0;
  // no order has more slices than 32768 = 64 groups of 16
  const int64_t s = std::min<int64_t>((nmax + FAR_SLICE - 1) / FAR_SLICE, 16);
  return 5 * N * s / 2048;
}

// Blocks of k_far (FAR_BLK threads each), which loop over the records: one a
// record up to FAR_GRID, far more than the GPU holds and far below the 2^32
// threads that a launch may have.
constexpr int FAR_BLK = 256;
constexpr int64_t FAR_GRID = 1 << 20;
static constexpr int64_t far_grid(int64_t records) { return records < FAR_GRID ? records : FAR_GRID; }

}  // namespace dpr1
