// Launch shapes that are chosen by the sizes of a call, apart from the kernels
// so that they can be checked on the host.
#pragma once

#include <cstdint>

namespace rbp {
namespace rules {

// ---- rb_push ------------------------------------------------------------------

constexpr int kPushThreads = 256;
constexpr int kPushLoads = 8;  // tokens a thread has in flight
constexpr int kPushTokens = kPushLoads * kPushThreads;  // of one pass of a block

// Blocks per new record, each taking every push_rows-th pass over it.  Two
// blocks per compute unit while there are few records; and, as a stretch of
// slot_tokens may be filled by one record of many short ones, enough that no
// block runs more than 8 passes (1.4 us each), up to 16: the blocks of short
// records that find no pass cost less than that.  512 records, one of 262144
// tokens among 100-token ones: 184 us with one block each, 16 with 16; 32768
// tokens each: 46.5 with one, 43.0 with two.
inline int64_t push_rows(int64_t n_new, int64_t slot_tokens) {
  const int64_t passes = (slot_tokens + kPushTokens - 1) / kPushTokens;
  const int64_t fill = 512 / n_new;
  int64_t rows = (passes + 7) / 8;
  if (rows > 16) rows = 16;
  if (rows < fill) rows = fill;
  return rows < passes ? rows : passes;
}

// ---- rb_sample_gather, packed -------------------------------------------------

constexpr int kFuseDraws = 512;     // draws that a block can redo, one per thread
constexpr int kPackedSmall = 512;   // threads of a block in windows of up to 2^17 positions
constexpr int kPackedLarge = 1024;  // and beyond: half as many blocks redo the draws

struct PackedRoute {
  int threads, positions;  // of the one launch's blocks and of a thread
  int64_t blocks;          // 0: the draws first, then the gather, in launches of their own
};

// Draw and gather in one launch, every block redoing all the draws, pays while
// the blocks run at once -- one per compute unit where slots are found by rank
// (the granules' offsets and masks in LDS and registers), two otherwise -- and
// the records that they read over and over stay few.  Two positions per thread
// halve the blocks once more.  Device times, one launch against two: 524288
// positions of 64 uniform draws 5.3 us against 6.6, of 512 7.4 / 8.0 (8.4 with
// one position per thread); 10^6 of 64 6.6 / 7.9; mix draws from 32768 records:
// 262144 positions of 512 draws 12.4 / 13.7, 2000000 of 24 in 977 blocks 41 / 15.5.
inline PackedRoute packed_route(int64_t n_draw, int64_t max_tokens, bool ranks) {
  const PackedRoute none{0, 0, 0};
  if (n_draw > kFuseDraws) return none;
  const auto blocks_of = [&](int64_t per) { return max_tokens / per + (max_tokens % per != 0); };
  if (max_tokens <= 256 * kPackedSmall) return {kPackedSmall, 1, blocks_of(kPackedSmall)};
  const int64_t at_once = ranks ? 256 : 512, one = blocks_of(kPackedLarge),
                two = blocks_of(2 * kPackedLarge);
  if (one <= at_once && one * n_draw <= 3 << 16) return {kPackedLarge, 1, one};
  if (two <= at_once && two * n_draw <= 1 << 17) return {kPackedLarge, 2, two};
  return none;
}

// ---- rb_sample_gather, padded -------------------------------------------------

constexpr int kDrawThreads = 1024;  // draws that one block can make

// Whether every block of a padded gather finds its row's draw by itself, in one
// launch.  Without ranks that is one Philox block.  With them each block scans
// the offsets of the table's n_granules granules (0: no ranks) or searches
// them, so for many draws from a large table a launch that makes the draws and
// one that copies are faster, unless the rows are long.  Device times, one
// launch against two, mix draws: 512 of 10^6 records 13.0 / 13.6 us, 600 15.8 /
// 14.2, 1024 19.2 / 16.9; 1024 of 3 * 10^6 30.4 / 24.3; 1024 rows of 1000 from
// 66000 records 18.5 / 18.8, of 100 16.5 / 15.4.
inline bool padded_one_launch(int64_t n_draw, int64_t l_max, int64_t n_granules) {
  if (n_draw > kDrawThreads) return false;
  if (n_granules == 0 || l_max > 2 * n_granules) return true;
  return n_draw <= (n_granules < 256 ? 768 : 512);
}

}  // namespace rules
}  // namespace rbp
