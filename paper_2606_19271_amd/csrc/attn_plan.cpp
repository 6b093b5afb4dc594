// attn_plan.cpp -- host-side sizes of the launches (grids, plan buffer, copy chunks), shared by
// the argument checks of ts_attn.cpp and the launch code; no device code.
#include <stdint.h>

#include <algorithm>

#include "attn_launch.h"

namespace tsattn {

int64_t packed_grid_bound(int32_t total_q, int32_t nseq, int32_t H, int32_t n_split) {
  // sum_s ceil(Lq_s / tile) <= ceil(Tq / tile) + nseq
  return (int64_t)H * n_split * (((int64_t)total_q + kQueryTile - 1) / kQueryTile + nseq);
}

int64_t packed_items(int32_t total_q, int32_t nseq, int32_t H, int32_t n_split, int32_t tile) {
  // ceil(x / tile) <= (x + tile - 1) / tile for every segment
  return (int64_t)H * n_split * (((int64_t)total_q + (int64_t)(tile - 1) * nseq) / tile);
}

// 64-query items as long as they all run at once: then the call takes one item's time, and an item
// takes 0.5 to 0.7 of a 256-query item's (measured, 1024 keys: 11.3 against 17.5 us for 16 heads at
// d = 64, 14.9 against 21.6 at d = 128; 256 keys x 4 heads 5.9 against 8.2 and 6.6 against 9.5).  In
// two rounds they lose: 18 heads 20.3 against 17.5 us and 26.1 against 21.6.  Up to 64 keys there is
// nothing to split (4.65 against 4.7 us at d = 64, 4.8 against 4.4 at d = 128).
bool small_items(int64_t items, int32_t max_k, int32_t cus) { return items <= cus && max_k > 64; }

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Estimated time (us) of a chunk call with n key ranges in 256- or 64-query items.  The lengths are on
// the device: the host knows the totals and the longest, and takes the segments as of average length.
// Constants: measured GPU times of 48 shapes, 1 to 16 ranges each, in both item sizes; over them the
// choice is 1.5 % slower than the best measured one (geometric mean; counting rounds of items alone:
// 16 %, for instance 4680 queries x 9360 keys x 12 heads 359 us in 10 ranges against 228 in one, and
// three 1560-query chunks x 12 heads 338 us unsplit against 240 in three ranges).
double split_time(const SplitShape& c, int32_t n, bool small, int32_t cus) {
  const int64_t kt = key_tile(c.d);
  const double avg_q = (double)c.total_q / c.nseq, avg_tiles = (double)c.total_k / c.nseq / kt;
  const int64_t range = ceil_div(ceil_div(c.max_k, kt), n);  // key tiles of the longest items
  double us;
  if (small) {  // only where all items run at once
    const int64_t items = (int64_t)c.H * c.nseq * ceil_div(ceil_div(c.total_q, c.nseq), kSmallTile) * n;
    if (!small_items(items, c.max_k, cus)) return 1e30;
    us = range * (c.d == 64 ? 0.7 : 0.57) + 4.5;
  } else {
    // a tile costs more with more CUs at work (LDS-DMA and power): at + with * (share of the CUs)
    const double at = c.d == 64 ? 1.55 : 1.05, with = c.d == 64 ? 0.4 : 0.5, item = 8;
    const int64_t full = (int64_t)avg_q / kQueryTile;
    const double rest = avg_q - (double)(full * kQueryTile);
    const double items = (double)c.H * c.nseq * n * (full + (rest == 0 ? 0 : rest <= 32 ? 0.6 : 1));
    const double rounds = items / cus;
    if (ceil_div(c.max_k, kt) * kt * c.nseq <= c.total_k * 1.05 + (double)kt * c.nseq) {
      // items of one length run in rounds
      const int64_t whole = (int64_t)rounds;
      const double last = rounds - (double)whole;
      us = whole * (range * (at + with) + item) + (last > 0 ? range * (at + with * last) + item : 0);
    } else {
      // longest first: the mean load, and about half an item where the CUs run out of work
      const double load = rounds * avg_tiles / n;
      const double tiles = std::max((double)range, load + 0.5 * range);
      us = tiles * (at + with * std::min(1.0, load / tiles)) + std::max(1.0, rounds) * item;
    }
  }
  // the merge: a launch, and the partials written and read at about 4 TB/s
  if (n > 1) us += 7 + (double)n * c.total_q * c.H * (4 * c.d + 4) / 4e6;
  return us;
}

}  // namespace

int32_t auto_splits(const SplitShape& c, int32_t max_n, int32_t cus) {
  const int64_t tiles = ceil_div(c.max_k, key_tile(c.d));
  int32_t best = 1;
  double best_us = 1e30;
  for (int32_t n = 1; n <= max_n && (n == 1 || tiles / n >= 4); ++n)
    for (int small = 0; small < 2; ++small) {
      const double us = split_time(c, n, small != 0, cus);
      if (us < best_us) { best_us = us; best = n; }
    }
  return best;
}

int64_t merge_blocks(int32_t total_q, int32_t H, int32_t d) {
  return ((int64_t)total_q * H * (d / 8) + kMergeThreads - 1) / kMergeThreads;
}

int64_t plan_ints(int32_t nseq) { return 2 + 2 * (int64_t)nseq; }

int64_t copy_chunk_bytes(bool src_host) { return src_host ? kHostReadChunkBytes : kCopyChunkBytes; }

}  // namespace tsattn
