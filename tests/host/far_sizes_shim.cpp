// C entry points over the sizes of the far-field expansions (far_sizes.h), for CPU tests.
#include "../../paper_1405_7537_amd/csrc/far_sizes.h"

extern "C" {
int64_t shim_far_blocks(int64_t n) {
  return dpr1::far_grid((n + dpr1::WAVE - 1) / dpr1::WAVE + dpr1::far_wide_records(n));
}
int64_t shim_far_records(int64_t n) { return dpr1::far_wide_records(n); }
int64_t shim_far_room(int64_t n) { return dpr1::far_wide_room(n); }
int64_t shim_far_min(void) { return dpr1::FAR_MIN; }
int64_t shim_far_batch_own(int64_t N, int64_t nmax, int64_t items) { return dpr1::far_batch_own(N, nmax, items); }
int64_t shim_far_batch_wide(int64_t N, int64_t nmax) { return dpr1::far_batch_wide(N, nmax); }
int64_t shim_far_block_threads(void) { return dpr1::FAR_BLK; }
}
