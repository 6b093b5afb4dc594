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
// nothing to split (4.65 against 4.7 us at d = 64, 4.8 against 4.4 at d = 128).  The items of a packed
// call are counted by packed_items from the totals alone, nearly one too many a segment, head and range, so
// a batch whose items would fit may still run in 256-query ones.
bool small_items(int64_t items, int32_t max_k, int32_t cus) { return items <= cus && max_k > 64; }

// A wave's own plan costs each round of items 0.085 us a segment, and saves the planning kernel, 4 to
// 7 us a call.  Measured over 2 to 64 segments and up to 40 rounds (us with the wave's plan and with the
// kernel's): 8 segments in 5 rounds 109.8 and 112.6, 12 in 7.5 167.9 and 168.8, 24 in 7.5 53.0 and
// 47.1, 64 in 10 115.8 and 60.0; the two meet at about 110 segments x rounds.
bool wave_plan(int32_t nseq, int64_t items, int32_t cus) {
  return nseq == 1 || (nseq <= kWavePlanSegs && nseq * std::max<int64_t>(items, cus) <= (int64_t)96 * cus);
}

int32_t auto_splits(int32_t total_q, int32_t max_k, int32_t H, int32_t d, int32_t cus) {
  const int64_t items = (int64_t)H * (((int64_t)total_q + kQueryTile - 1) / kQueryTile);
  const int64_t tiles = ((int64_t)max_k + key_tile(d) - 1) / key_tile(d);
  if (items <= 0 || items >= cus || tiles < 8) return 1;
  int32_t best = 1;
  int64_t best_cost = INT64_MAX;
  for (int32_t n = 1; n <= kMaxSplits && tiles / n >= 4; ++n) {
    const int64_t cost = (items * n + cus - 1) / cus * ((tiles + n - 1) / n);
    if (cost < best_cost) { best_cost = cost; best = n; }
  }
  return best;
}

int64_t merge_blocks(int32_t total_q, int32_t H, int32_t d) {
  return ((int64_t)total_q * H * (d / 8) + kMergeThreads - 1) / kMergeThreads;
}

int64_t plan_ints(int32_t nseq) { return 2 + 2 * (int64_t)nseq; }

int64_t copy_chunk_bytes(bool src_host) { return src_host ? kHostReadChunkBytes : kCopyChunkBytes; }

// Up to 128 MiB, read and written 256 MiB, the Infinity Cache holds a copy for the call that reads it
// next.  Copy alone, and with attention over the copied keys and values after it (us, plain and
// non-temporal): 40 MiB 13.1 and 14.5, 46.4 and 51.7; 96 MiB 29.5 and 32.6, 80.7 and 89.8; 128 MiB 39.0
// and 43.5, 103.6 and 113.5; 160 MiB 59.2 and 54.2, 124.6 and 134.4; 256 MiB 92.9 and 86.7, 209 and 203.
bool bypass_caches(int64_t bytes) { return bytes > (int64_t)128 << 20; }

}  // namespace tsattn
