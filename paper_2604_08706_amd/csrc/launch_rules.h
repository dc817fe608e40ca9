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

}  // namespace rules
}  // namespace rbp
