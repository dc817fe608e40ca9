// Marked slots of a record table, found by rank.
//
// Slots are marked in 64-bit masks and counted per granule of 1024; a count
// carries two numbers, the marked slots in its low 32 bits and above them the
// slots tied for the last places (selection without replacement: keys equal to
// the last one that is taken), of which the first `need` in slot order count.
// Finding the k-th by rank takes a search over the granules' offsets and one
// granule's masks, where a compacted list of slots takes a pass that writes it
// and, before that, a scan of its own.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rbp {
namespace ranks {

constexpr int kGranule = 1024;         // slots per count
constexpr int kWords = kGranule / 64;  // masks per granule

struct View {
  const uint64_t *mark, *tie;  // [nb * kWords], 16-byte aligned; tie may be null
  const int64_t* off;          // [nb], counts before each granule
  int32_t nb;
  int64_t need, n;  // n: slots that have a rank
};

// Ranks in front of a granule with offset (or total) `packed`.
__host__ __device__ __forceinline__ int64_t below(int64_t packed, int64_t need) {
  const int64_t ties = packed >> 32;
  return (packed & 0xffffffffll) + (ties < need ? ties : need);
}

// Position of the k-th set bit of m (k < its bits).
__host__ __device__ __forceinline__ int32_t kth_bit(uint64_t m, int32_t k) {
  int32_t at = 0;
#pragma unroll
  for (int half = 32; half >= 1; half >>= 1) {
    const int32_t c = __builtin_popcountll(m & ((1ull << half) - 1ull));
    if (k >= c) {
      k -= c;
      m >>= half;
      at += half;
    }
  }
  return at;
}

// The slot of rank k (0 <= k < n), slots ascending.
__host__ __device__ __forceinline__ int64_t slot_of(const View& v, int64_t k) {
  int32_t lo = 0, hi = v.nb;  // the last granule with at most k ranks in front
  while (hi - lo > 1) {
    const int32_t m = (lo + hi) >> 1;
    if (below(v.off[m], v.need) <= k) lo = m; else hi = m;
  }
  // the granule's masks in one go (16-byte loads), then no more memory
  uint64_t m[kWords];
  const ulonglong2* mark = reinterpret_cast<const ulonglong2*>(v.mark + (int64_t)lo * kWords);
#pragma unroll
  for (int w = 0; w < kWords; w += 2) {
    const ulonglong2 x = mark[w / 2];
    m[w] = x.x;
    m[w + 1] = x.y;
  }
  // ties are rare (the one key of 63 random bits that is taken last, mostly):
  // only a granule that has some, or the last one, reads their masks.  Drawing
  // 1024 of 3 million records so takes 95.8 us, with all of them read 100.4.
  const int64_t o = v.off[lo], ties = o >> 32;
  if (v.tie != nullptr && (lo + 1 == v.nb || (v.off[lo + 1] >> 32) != ties)) {
    const ulonglong2* tie = reinterpret_cast<const ulonglong2*>(v.tie + (int64_t)lo * kWords);
    int64_t allow = v.need - (ties < v.need ? ties : v.need);
#pragma unroll
    for (int w = 0; w < kWords; w += 2) {
      const ulonglong2 x = tie[w / 2];
      uint64_t t[2] = {x.x, x.y};
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int32_t c = __builtin_popcountll(t[i]);
        if (c == 0) continue;
        if (allow < c)  // keep the first `allow` of them
          t[i] = allow == 0 ? 0ull : t[i] & (~0ull >> (63 - kth_bit(t[i], (int32_t)allow - 1)));
        m[w + i] |= t[i];
        allow -= allow < c ? allow : c;
      }
    }
  }
  int32_t rem = (int32_t)(k - below(o, v.need)), word = 0;
  uint64_t at = m[0];
  bool found = false;
#pragma unroll
  for (int w = 0; w < kWords; ++w) {
    const int32_t c = __builtin_popcountll(m[w]);
    if (!found && rem < c) {
      found = true;
      word = w;
      at = m[w];
    }
    if (!found) rem -= c;
  }
  return ((int64_t)lo * kWords + word) * 64 + (found ? kth_bit(at, rem) : 0);
}

}  // namespace ranks
}  // namespace rbp
