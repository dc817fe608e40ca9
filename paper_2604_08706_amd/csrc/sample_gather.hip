// Replay-buffer sampling and batch gather (rb_sample_gather).
//
// Paper: the buffer is a FIFO list whose sampling does not remove records
// (Sec. 3.1; App. B "BufferStructure"); draws are uniform with replacement
// (Sec. 4); positive-bias retention keeps the freshest (1-delta)N rollouts
// plus the freshest delta*N correct rollouts older than those (Sec. 5;
// App. D.4).  The positive-prioritised mixture is an addition (see header).
//
// Device pipeline (one stream):
//   [mix/retain only] pos_mask : one bit per slot, set for positives, and
//       their number per granule of 1024 slots;
//   [without replacement] slot_key -> select_cand -> select_rest : an MSD radix
//       select (8-bit digits) finds the n_draw-th smallest 64-bit slot key K
//       exactly -- the top digit from per-block histograms of every key, the
//       seven lower ones by every block over the keys that share the top
//       digit -- and marks the slots with a key below K and those equal to K,
//       again one bit per slot with the numbers per granule;
//   the k-th marked slot (slot = FIFO position, 0 = oldest) is then found by
//   rank (ranks.h): no list of slots is written or read back.
//   up to 1024 draws, as far as it pays (launch_rules.h), one launch:
//   sample_packed / sample_padded : every block draws what it copies --
//       Philox4x64-10 block -> slot -> record -- and, packed, scans all the
//       lengths; the first block writes the per-draw outputs;
//   otherwise
//   draw     : one thread per draw, per-draw outputs; scan of lengths ->
//              cu_seqlens, n_tokens (one block up to 1024 draws, else
//              draw_rows -> draw_scan -> draw_cu);
//   gather   : one block column per draw (packed: the part of its sequence
//              inside the window; padded: its l_max row); coalesced copies
//              from the token arena.
// Everything is integer work or a bit-exact copy of stored floats.

#include <atomic>
#include <mutex>

#include "launch_rules.h"
#include "ranks.h"
#include "rbp_internal.h"

namespace {

using rbp::ranks::kGranule;
using rbp::ranks::kWords;
using rbp::ranks::View;

constexpr int kMaskThreads = 256;
constexpr int kLdsGranules = 2048;     // granules whose offsets a block scans itself
constexpr int kFuseThreads = 256;      // of the padded kernels
using rbp::rules::kFuseDraws;          // draws that sample_packed redoes in every block
constexpr int kRowVecs = 4;            // 16-byte groups of a padded row per thread
constexpr int kRowSingles = 8;         // or positions, where rows are not aligned to them
using rbp::rules::kDrawThreads;     // single-block draw pass, up to this many draws
constexpr int kRowThreads = 256;    // draws per block beyond that
constexpr int kMaxRowBlocks = (1 << 20) / kRowThreads;

// ---- Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11) ----------------------
struct Block4 {
  uint64_t x0, x1, x2, x3;
};

__device__ __forceinline__ Block4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2,
                                                uint64_t c3, uint64_t k0, uint64_t k1) {
  const uint64_t kMul0 = 0xD2E7470EE14C6C93ull, kMul1 = 0xCA5A826395121157ull;
  const uint64_t kWeyl0 = 0x9E3779B97F4A7C15ull, kWeyl1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += kWeyl0;
      k1 += kWeyl1;
    }
    const uint64_t hi0 = __umul64hi(kMul0, c0), lo0 = kMul0 * c0;
    const uint64_t hi1 = __umul64hi(kMul1, c2), lo1 = kMul1 * c2;
    const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  return {c0, c1, c2, c3};
}

__device__ __forceinline__ int64_t phys_row(int64_t slot, int64_t head, int64_t cap) {
  int64_t r = head + slot;
  return r >= cap ? r - cap : r;
}

// Block-wide exclusive scan of one int64 per thread (fixed order).
template <int NT>
__device__ int64_t block_exclusive_scan(int64_t v, int64_t* total, int64_t* lds_waves) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int64_t o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) lds_waves[wave] = incl;
  __syncthreads();
  int64_t wave_base = 0, sum = 0;
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wave) wave_base += lds_waves[w];
    sum += lds_waves[w];
  }
  __syncthreads();
  *total = sum;
  return wave_base + incl - v;
}

// ---- ranks of marked slots (ranks.h) -----------------------------------------

// Where a launch finds the marks: masks and counts per granule, and, for
// tables of more than kLdsGranules granules, their scanned offsets and total.
struct Ranks {
  const uint64_t *mark, *tie;  // [nb * kWords]; tie may be null
  const int64_t* counts;       // [nb]
  const int64_t* offsets;      // [nb], or null: scanned by each block
  const int64_t* total;        // with offsets
  const int64_t* need;         // ties to take, in slot order (with tie)
  int32_t nb;
};

// Offsets of the granules (scanned into `off_s` unless they are given) and the
// number of ranks.
template <int NT>
__device__ View view_ranks(const Ranks& r, int64_t (&off_s)[kLdsGranules], int64_t* lds_waves) {
  View v{r.mark, r.tie, r.offsets, r.nb, r.tie != nullptr ? *r.need : 0, 0};
  if (r.offsets != nullptr) {
    v.n = rbp::ranks::below(*r.total, v.need);
    return v;
  }
  constexpr int kPer = kLdsGranules / NT;
  const int32_t per = (r.nb + NT - 1) / NT;  // <= kPer
  const int32_t lo = (int32_t)threadIdx.x * per;
  int64_t c[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    c[k] = k < per && lo + k < r.nb ? r.counts[lo + k] : 0;
    sum += c[k];
  }
  int64_t total;
  int64_t at = block_exclusive_scan<NT>(sum, &total, lds_waves);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (k < per && lo + k < r.nb) off_s[lo + k] = at;
    at += c[k];
  }
  __syncthreads();
  v.off = off_s;
  v.n = rbp::ranks::below(total, v.need);
  return v;
}

// Positives of granule b among the slots [0, n_range).
__global__ void __launch_bounds__(kMaskThreads) pos_mask_kernel(
    const float* __restrict__ reward, int64_t head, int64_t cap, int64_t n_range,
    uint64_t* __restrict__ mark, int64_t* __restrict__ counts) {
  __shared__ int32_t part[kMaskThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kPer = kGranule / kMaskThreads;  // words per wave
  const int64_t w0 = (int64_t)blockIdx.x * kWords + wave * kPer;
  float x[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int64_t s = (w0 + k) * 64 + lane;
    x[k] = s < n_range ? reward[phys_row(s, head, cap)] : 0.0f;
  }
  int32_t c = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint64_t m = __ballot(x[k] > 0.0f);
    if (lane == 0) mark[w0 + k] = m;
    c += __popcll(m);
  }
  if (lane == 0) part[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t n = 0;
    for (int w = 0; w < kMaskThreads / 64; ++w) n += part[w];
    counts[blockIdx.x] = n;
  }
}

// Offsets and total of the counts, for tables of more than kLdsGranules
// granules.
__global__ void __launch_bounds__(1024) rank_scan_kernel(const int64_t* __restrict__ counts,
                                                         int64_t* __restrict__ offsets, int64_t nb,
                                                         int64_t* __restrict__ total_out) {
  __shared__ int64_t lds[1024 / 64];
  int64_t carry = 0;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t v = i < nb ? counts[i] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<1024>(v, &total, lds);
    if (i < nb) offsets[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) *total_out = carry;
}

// ---- selection without replacement -----------------------------------------

constexpr int kKeyBlocks = 256;   // key kernel blocks (at most): key segments; a power of 2
constexpr int kKeyThreads = 1024;
constexpr int kRestThreads = 1024;
constexpr int kRestRegKeys = 16;  // candidates per thread held in registers

// Radix-select state: the key digits fixed so far and how many keys still to
// be taken among those sharing them.
struct SelState {
  uint64_t prefix;
  int64_t need;
};

// Key segment b of n keys split over n_seg blocks: [b * per, min(n, (b+1) * per)).
__device__ __forceinline__ int64_t seg_len(int64_t n, int64_t n_seg) {
  return (n + n_seg - 1) / n_seg;
}

// Key of slot s: the top 63 bits of word 0 of the Philox block with counter
// (s, step, 1, 0); for never-used-first, bit 63 set when the slot was used.
// Block b keys segment b and writes the histogram of the top digit (bits
// 56..63) of its keys to row b of `top_hist`: no global atomics, so the 256
// bins are not contended by every block.
__global__ void __launch_bounds__(kKeyThreads) slot_key_kernel(
    uint64_t seed, uint64_t step, int64_t n_live, int64_t head, int64_t cap,
    const int32_t* __restrict__ use_count, uint64_t* __restrict__ keys,
    uint32_t* __restrict__ top_hist) {
  __shared__ uint32_t h[256];
  if (threadIdx.x < 256) h[threadIdx.x] = 0u;
  __syncthreads();
  const int64_t per = seg_len(n_live, gridDim.x);
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < n_live ? lo + per : n_live;
  for (int64_t s = lo + threadIdx.x; s < hi; s += kKeyThreads) {
    uint64_t k = philox4x64_10((uint64_t)s, step, 1, 0, seed, 0).x0 >> 1;
    if (use_count != nullptr && use_count[phys_row(s, head, cap)] > 0) k |= 1ull << 63;
    keys[s] = k;
    atomicAdd(&h[k >> 56], 1u);
  }
  __syncthreads();
  if (threadIdx.x < 256) top_hist[blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// Bin t of the block holding the need-th smallest remaining key: the one
// thread whose exclusive prefix is below `need` and inclusive prefix reaches
// it (empty bins never qualify).
__device__ __forceinline__ bool holds_need(int64_t excl, int64_t count, int64_t need) {
  return excl < need && need <= excl + count;
}

// Every block sums the per-segment top-digit histograms (four threads per
// bin) and picks the top digit; the first one keeps it.  Block b then lists
// the keys of segment b whose top digit is the selected one at the start of
// the segment's stretch of `cand` (order free: only their digit histograms
// are taken), and their number in cand_cnt[b].  One LDS atomic per wave, no
// global ones.
__global__ void __launch_bounds__(kKeyThreads) select_cand_kernel(
    const uint64_t* __restrict__ keys, int64_t n, const uint32_t* __restrict__ top_hist,
    int64_t n_draw, SelState* __restrict__ st, uint64_t* __restrict__ cand,
    uint32_t* __restrict__ cand_cnt) {
  __shared__ uint32_t part[kKeyThreads / 256][256];
  __shared__ int64_t lds[kKeyThreads / 64];
  __shared__ uint32_t cnt, s_top;
  const int32_t n_seg = (int32_t)gridDim.x;
  const int bin = threadIdx.x & 255, q = threadIdx.x >> 8;
  uint32_t c = 0u;
#pragma unroll 8
  for (int32_t b = q; b < n_seg; b += kKeyThreads / 256) c += top_hist[b * 256 + bin];
  part[q][bin] = c;
  if (threadIdx.x == 0) cnt = 0u;
  __syncthreads();
  int64_t v = 0;
  if (threadIdx.x < 256)
    for (int i = 0; i < kKeyThreads / 256; ++i) v += part[i][bin];
  int64_t total;
  const int64_t excl = block_exclusive_scan<kKeyThreads>(v, &total, lds);
  if (threadIdx.x < 256 && holds_need(excl, v, n_draw)) {
    s_top = (uint32_t)bin;
    if (blockIdx.x == 0) {
      st->prefix = (uint64_t)bin << 56;
      st->need = n_draw - excl;
    }
  }
  __syncthreads();
  const uint64_t top = s_top;
  const int lane = threadIdx.x & 63;
  const int64_t per = seg_len(n, gridDim.x);
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < n ? lo + per : n;
  for (int64_t base = lo; base < hi; base += kKeyThreads) {
    const int64_t s = base + threadIdx.x;
    const uint64_t k = s < hi ? keys[s] : 0ull;
    const bool take = s < hi && (k >> 56) == top;
    const uint64_t m = __ballot(take);
    if (m == 0ull) continue;
    uint32_t at = 0u;
    if (lane == 0) at = atomicAdd(&cnt, (uint32_t)__popcll(m));
    at = __shfl(at, 0, 64);
    if (take) cand[lo + at + __popcll(m & ((1ull << lane) - 1ull))] = k;
  }
  __syncthreads();
  if (threadIdx.x == 0) cand_cnt[blockIdx.x] = cnt;
}

// One block's search for the exact n_draw-th smallest key: the lower digits,
// most significant first, over the candidates only (the first kRestThreads *
// kRestRegKeys of them held in registers, any further ones re-read each pass),
// until at most kRestThreads keys share the prefix; those are then ranked
// directly, each thread counting the survivors below and up to its own.
// Integer counts only: the result does not depend on the order of any
// addition.  Returns the key and the number of its ties to be taken.
__device__ SelState select_rest(const uint64_t* __restrict__ cand,
                                const uint32_t* __restrict__ cand_cnt, int32_t n_seg, int64_t n,
                                const SelState& top) {
  __shared__ uint32_t h[256];
  __shared__ int64_t lds[kRestThreads / 64];
  __shared__ int64_t seg_start[kKeyBlocks + 1];
  __shared__ uint64_t surv[kRestThreads];
  __shared__ uint64_t s_prefix;
  __shared__ int64_t s_need, s_match;
  __shared__ uint32_t s_surv;
  const int64_t c = threadIdx.x < n_seg ? (int64_t)cand_cnt[threadIdx.x] : 0;
  int64_t nc;
  const int64_t excl = block_exclusive_scan<kRestThreads>(c, &nc, lds);
  if (threadIdx.x < n_seg) seg_start[threadIdx.x] = excl;
  if (threadIdx.x == 0) {
    seg_start[n_seg] = nc;
    s_surv = 0u;
  }
  __syncthreads();
  const int64_t per = seg_len(n, n_seg);
  // candidate i (< nc) sits at entry i - seg_start[b] of segment b, the last
  // segment starting at or before i
  // (a fixed eight halvings over n_seg <= kKeyBlocks = 256 starts, so the
  // searches of a thread's candidates interleave)
  auto cand_pos = [&](int64_t i) {
    int lo = 0;
#pragma unroll
    for (int step = kKeyBlocks / 2; step > 0; step >>= 1) {
      const int m = lo + step;
      if (m < n_seg && seg_start[m] <= i) lo = m;
    }
    return lo * per + (i - seg_start[lo]);
  };
  // positions first, then all the loads together (nc >= 1: the selected
  // bucket holds the need-th key; indices past it re-read the last one),
  // in as many rounds of four as the candidates fill
  uint64_t reg[kRestRegKeys];
#pragma unroll
  for (int u0 = 0; u0 < kRestRegKeys; u0 += 4) {
    if ((int64_t)u0 * kRestThreads >= nc) break;
    int64_t at[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = threadIdx.x + (int64_t)(u0 + u) * kRestThreads;
      at[u] = cand_pos(i < nc ? i : nc - 1);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) reg[u0 + u] = cand[at[u]];
  }
  // calls f(k) for every candidate k
  auto each_cand = [&](auto&& f) {
#pragma unroll
    for (int u = 0; u < kRestRegKeys; ++u)
      if (threadIdx.x + (int64_t)u * kRestThreads < nc) f(reg[u]);
    for (int64_t i = threadIdx.x + (int64_t)kRestRegKeys * kRestThreads; i < nc;
         i += kRestThreads)
      f(cand[cand_pos(i)]);
  };
  uint64_t prefix = top.prefix;
  int64_t need = top.need;
  int64_t n_match = nc;  // keys sharing the digits fixed so far
  int shift = 56;        // the prefix fixes the bits from `shift` up
  while (shift > 0 && n_match > kRestThreads) {
    shift -= 8;
    if (threadIdx.x < 256) h[threadIdx.x] = 0u;
    __syncthreads();
    const uint64_t hi = prefix >> (shift + 8);
    each_cand([&](uint64_t k) {
      if ((k >> (shift + 8)) == hi) atomicAdd(&h[(k >> shift) & 255u], 1u);
    });
    __syncthreads();
    const int64_t v = threadIdx.x < 256 ? (int64_t)h[threadIdx.x] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<kRestThreads>(v, &total, lds);
    if (threadIdx.x < 256 && holds_need(ex, v, need)) {
      s_prefix = prefix | ((uint64_t)threadIdx.x << shift);
      s_need = need - ex;
      s_match = v;
    }
    __syncthreads();
    prefix = s_prefix;
    need = s_need;
    n_match = s_match;
  }
  if (shift > 0) {
    // at most kRestThreads survivors: list them (order free), then the one
    // with `need - 1` survivors strictly below it and at least `need` up to
    // it is the key; equal keys all write the same values
    const uint64_t hi = prefix >> shift;
    each_cand([&](uint64_t k) {
      if ((k >> shift) == hi) {
        const uint32_t i = atomicAdd(&s_surv, 1u);  // < n_match <= kRestThreads
        if (i < kRestThreads) surv[i] = k;
      }
    });
    __syncthreads();
    if (threadIdx.x < n_match) {
      const uint64_t mine = surv[threadIdx.x];
      int32_t less = 0, leq = 0;
#pragma unroll 4
      for (int32_t i = 0; i < (int32_t)n_match; ++i) {
        const uint64_t o = surv[i];
        less += o < mine;
        leq += o <= mine;
      }
      if (less < need && need <= leq) {
        s_prefix = mine;
        s_need = need - less;
      }
    }
    __syncthreads();
    prefix = s_prefix;
    need = s_need;
  }
  return SelState{prefix, need};
}

// Marks the slots with a key below the n_draw-th smallest key K and those
// equal to it (ties).  Every block finds K itself (select_rest: a few us,
// where a launch of one block for it and the wait for its result cost 11);
// the first one keeps the number of ties to be taken.  One granule per block
// and round, 64 slots per wave.
__global__ void __launch_bounds__(kRestThreads) select_rest_kernel(
    const uint64_t* __restrict__ keys, int64_t n, const SelState* __restrict__ top,
    const uint64_t* __restrict__ cand, const uint32_t* __restrict__ cand_cnt, int32_t n_seg,
    int32_t nb, uint64_t* __restrict__ mark, uint64_t* __restrict__ tie,
    int64_t* __restrict__ counts, int64_t* __restrict__ need) {
  static_assert(kRestThreads == kGranule, "one slot per thread and round");
  __shared__ int64_t part[kWords];
  const SelState sel = select_rest(cand, cand_cnt, n_seg, n, *top);
  if (blockIdx.x == 0 && threadIdx.x == 0) *need = sel.need;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int32_t b = (int32_t)blockIdx.x; b < nb; b += (int32_t)gridDim.x) {
    const int64_t s = (int64_t)b * kGranule + threadIdx.x;
    const uint64_t k = s < n ? keys[s] : ~0ull;
    const uint64_t m = __ballot(s < n && k < sel.prefix);
    const uint64_t t = __ballot(s < n && k == sel.prefix);
    if (lane == 0) {
      mark[(int64_t)b * kWords + wave] = m;
      tie[(int64_t)b * kWords + wave] = t;
      part[wave] = (int64_t)__popcll(m) + ((int64_t)__popcll(t) << 32);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t sum = 0;
      for (int w = 0; w < kWords; ++w) sum += part[w];
      counts[b] = sum;
    }
    __syncthreads();
  }
}

struct DrawParams {
  int32_t mode, layout;
  uint64_t seed, step, p_q32;
  int64_t n_draw, n_live, head, cap;
  int64_t first_fresh, n_pos_keep;
  int32_t cur_version;
  int64_t max_tokens, token_begin, l_max;
};

// Per-call constants of the draws: the positives (slots with a rank), the
// retained positives and the size of the retained set.
struct DrawSet {
  int64_t n_pos, keep, n_set;
};

__device__ __forceinline__ DrawSet draw_set(const DrawParams& p, const View& v) {
  DrawSet d;
  d.n_pos = (p.mode == RB_POS_MIX || p.mode == RB_POS_RETAIN) ? v.n : 0;
  // retained set: the newest `keep` positives older than the fresh part, then
  // the fresh part [first_fresh, n_live)
  d.keep = d.n_pos < p.n_pos_keep ? d.n_pos : p.n_pos_keep;
  d.n_set = d.keep + (p.n_live - p.first_fresh);
  return d;
}

// Slot of draw j: the Philox4x64-10 block with counter (j, step, 0, 0) picks
// it (or the j-th selected slot without replacement).
template <bool kRanks>
__device__ __forceinline__ int64_t draw_slot(const DrawParams& p, const DrawSet& d,
                                             const View& v, int64_t j) {
  if constexpr (!kRanks)
    return (int64_t)__umul64hi(philox4x64_10((uint64_t)j, p.step, 0, 0, p.seed, 0).x0,
                               (uint64_t)p.n_live);
  if (p.mode == RB_NO_REPLACE || p.mode == RB_UNUSED_FIRST) return rbp::ranks::slot_of(v, j);
  const Block4 b = philox4x64_10((uint64_t)j, p.step, 0, 0, p.seed, 0);
  if (p.mode == RB_UNIFORM) return (int64_t)__umul64hi(b.x0, (uint64_t)p.n_live);
  int64_t k;  // rank of a positive
  if (p.mode == RB_POS_MIX) {
    if (d.n_pos == 0 || (b.x1 >> 32) >= p.p_q32)
      return (int64_t)__umul64hi(b.x0, (uint64_t)p.n_live);
    k = (int64_t)__umul64hi(b.x0, (uint64_t)d.n_pos);
  } else {
    if (d.n_set <= 0) return 0;
    const int64_t i = (int64_t)__umul64hi(b.x0, (uint64_t)d.n_set);
    if (i >= d.keep) return p.first_fresh + (i - d.keep);
    k = d.n_pos - d.keep + i;
  }
  return rbp::ranks::slot_of(v, k);
}

// The record table as the draws read it, and the outputs they write.
struct DrawTable {
  const int32_t* length;
  const float* advantage;
  const int32_t* version;
  const int64_t* arena_off;
  const int32_t* arena_tokens;
  const float* arena_old;
  int32_t* out_idx;
  float* out_adv;
  int32_t *out_len, *out_age, *cu_seqlens;
  int32_t* tokens;
  float* old_logp;
  int32_t* seq;
  int64_t* n_tokens;
};

// Per-draw outputs of draw j of slot `slot`, row r, length len.
__device__ __forceinline__ void write_draw(const DrawParams& p, const DrawTable& t, int64_t j,
                                           int64_t slot, int64_t r, int64_t len) {
  t.out_idx[j] = (int32_t)slot;
  t.out_adv[j] = t.advantage[r];
  t.out_len[j] = (int32_t)len;
  t.out_age[j] = p.cur_version - t.version[r];
}

// Its contribution to the stream (full length packed, min(length, l_max)
// padded).
__device__ __forceinline__ int64_t stream_len(const DrawParams& p, int64_t len) {
  return p.layout == RB_LAYOUT_PACKED ? len : (len < p.l_max ? len : p.l_max);
}

template <bool kRanks>
__device__ __forceinline__ int64_t draw_one(const DrawParams& p, const DrawSet& d,
                                            const View& v, const DrawTable& t, int64_t j) {
  const int64_t slot = draw_slot<kRanks>(p, d, v, j);
  const int64_t r = phys_row(slot, p.head, p.cap);
  const int64_t len = t.length[r];
  write_draw(p, t, j, slot, r, len);
  return stream_len(p, len);
}

__device__ __forceinline__ int64_t window_tokens(const DrawParams& p, int64_t sum) {
  if (p.layout != RB_LAYOUT_PACKED) return sum;
  const int64_t v = sum - p.token_begin;
  return v < 0 ? 0 : (v > p.max_tokens ? p.max_tokens : v);
}

__device__ __forceinline__ void write_totals(const DrawParams& p, int64_t sum,
                                             int64_t* __restrict__ n_tokens,
                                             int64_t* __restrict__ stream_total) {
  *n_tokens = window_tokens(p, sum);
  *stream_total = sum;
}

// ---- draw and gather in one launch ------------------------------------------
//
// A draw kernel and a gather kernel after it are two chains of dependent loads
// (draw: record; gather: draw, arena offset, tokens) and two launches, about
// 5 us each for the few draws of a training batch.  Here every block redoes the
// draws it needs -- one Philox block and two loads per draw -- so nothing is
// handed over; see launch_rules.h for where redoing the draws stops paying.

// Block b copies kThreads * kPos window positions, from b of those on; a thread
// makes one draw and copies kPos positions.  (Two draws and four positions a
// thread, in blocks of 256, are as many chains of loads one after another:
// 16384 positions of 512 mix draws from 32768 records took 13.0 us, now 10.8;
// 358400 of 512 uniform draws 9.2, the two launches 7.7.)
// kRanks: every mode but the uniform one, which needs none of the ranks'
// registers and LDS.
template <bool kRanks, int kThreads, int kPos>
__global__ void __launch_bounds__(kThreads) sample_packed_kernel(DrawParams p, Ranks ranks,
                                                                 DrawTable t) {
  static_assert(kThreads >= kFuseDraws, "one draw per thread");
  __shared__ int64_t off_s[kRanks ? kLdsGranules : 1];
  __shared__ int64_t lds[kThreads / 64];
  __shared__ int64_t src_s[kFuseDraws];     // arena offset of draw j
  __shared__ int32_t cu_s[kFuseDraws + 1];  // its stream position
  View v{};
  if constexpr (kRanks) v = view_ranks<kThreads>(ranks, off_s, lds);
  const DrawSet d = draw_set(p, v);
  const int64_t j = threadIdx.x;
  int64_t len = 0;
  if (j < p.n_draw) {
    const int64_t slot = draw_slot<kRanks>(p, d, v, j);
    const int64_t r = phys_row(slot, p.head, p.cap);
    len = t.length[r];
    src_s[j] = t.arena_off[r];
    if (blockIdx.x == 0) write_draw(p, t, j, slot, r, len);
  }
  int64_t total;
  const int64_t at = block_exclusive_scan<kThreads>(len, &total, lds);
  if (j < p.n_draw) {
    cu_s[j] = (int32_t)at;
    if (blockIdx.x == 0) t.cu_seqlens[j] = (int32_t)at;
  }
  if (j == 0) {
    cu_s[p.n_draw] = (int32_t)total;
    if (blockIdx.x == 0) {
      t.cu_seqlens[p.n_draw] = (int32_t)total;
      *t.n_tokens = window_tokens(p, total);
    }
  }
  __syncthreads();
  const int64_t w0 = (int64_t)blockIdx.x * (kThreads * kPos) + threadIdx.x;
  int32_t tk[kPos], sq[kPos];
  float ol[kPos];
#pragma unroll
  for (int k = 0; k < kPos; ++k) {  // all loads in flight before the first store
    const int64_t w = w0 + k * kThreads, pos = p.token_begin + w;
    tk[k] = 0;
    ol[k] = 0.0f;
    sq[k] = -1;
    if (w >= p.max_tokens || pos >= total) continue;
    int32_t lo = 0, hi = (int32_t)p.n_draw;  // the draw that holds pos
    while (hi - lo > 1) {
      const int32_t m = (lo + hi) >> 1;
      if (cu_s[m] <= pos) lo = m; else hi = m;
    }
    const int64_t src = src_s[lo] + (pos - cu_s[lo]);
    tk[k] = t.arena_tokens[src];
    ol[k] = t.arena_old[src];
    sq[k] = lo;
  }
#pragma unroll
  for (int k = 0; k < kPos; ++k) {
    const int64_t w = w0 + k * kThreads;
    if (w >= p.max_tokens) continue;
    t.tokens[w] = tk[k];
    t.old_logp[w] = ol[k];
    t.seq[w] = sq[k];
  }
}

// Row j of [n_draw, l_max] from the record at `off` of length n (clamped to
// l_max): positions past n hold token 0, log-prob 0, seq -1.  kVec: four
// positions per thread with 16-byte stores (l_max % 4 == 0, rows 16-byte
// aligned); the arena is read with 4-byte loads, its rows start anywhere.  A
// thread has kGroups groups (or positions) in flight.  The padding is set first
// and the loads are under one condition: as selects, which become two branches
// each, with the stride read from the launch, 4096 rows of 512 took 18.8 us
// and not 18.5, 100 rows of 16383 9.5 and not 7.5.  kSelect: behind a draw by
// rank it is the other way round, and the draws there are many and narrow: 1000
// rows of 1047 15.9 us as selects and 16.6 under one condition, 1024 rows of 400
// 15.5 and 15.9 (only wide ragged rows lose: 256 of 8191 16.1 and 15.1).
template <bool kVec, int kGroups, bool kSelect>
__device__ __forceinline__ void fill_row(int64_t j, int64_t l_max, int64_t n, int64_t off,
                                         const int32_t* __restrict__ arena_tokens,
                                         const float* __restrict__ arena_old,
                                         int32_t* __restrict__ tokens,
                                         float* __restrict__ old_logp,
                                         int32_t* __restrict__ seq) {
  int32_t* tok_row = tokens + j * l_max;
  float* old_row = old_logp + j * l_max;
  int32_t* seq_row = seq + j * l_max;
  if constexpr (kVec) {
    const int64_t step = (kSelect ? (int64_t)blockDim.x : kFuseThreads) * 4;
    for (int64_t p0 = blockIdx.y * (step * kGroups) + threadIdx.x * 4; p0 < l_max;
         p0 += gridDim.y * (step * kGroups)) {
      int32_t tk[kGroups][4], sq[kGroups][4];
      float ol[kGroups][4];
#pragma unroll
      for (int u = 0; u < kGroups; ++u)  // all loads in flight before the first store
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int64_t p = p0 + u * step + i;
          if constexpr (kSelect) {
            tk[u][i] = p < n ? arena_tokens[off + p] : 0;
            ol[u][i] = p < n ? arena_old[off + p] : 0.0f;
            sq[u][i] = p < n ? (int32_t)j : -1;
          } else {
            tk[u][i] = 0;
            ol[u][i] = 0.0f;
            sq[u][i] = -1;
            if (p < n) {
              tk[u][i] = arena_tokens[off + p];
              ol[u][i] = arena_old[off + p];
              sq[u][i] = (int32_t)j;
            }
          }
        }
#pragma unroll
      for (int u = 0; u < kGroups; ++u) {
        const int64_t p = p0 + u * step;
        if (kGroups > 1 && p >= l_max) continue;
        *reinterpret_cast<int4*>(tok_row + p) = make_int4(tk[u][0], tk[u][1], tk[u][2], tk[u][3]);
        *reinterpret_cast<float4*>(old_row + p) =
            make_float4(ol[u][0], ol[u][1], ol[u][2], ol[u][3]);
        *reinterpret_cast<int4*>(seq_row + p) = make_int4(sq[u][0], sq[u][1], sq[u][2], sq[u][3]);
      }
    }
  } else {
    const int64_t step = kSelect ? (int64_t)blockDim.x : kFuseThreads;
    for (int64_t p0 = blockIdx.y * (step * kGroups) + threadIdx.x; p0 < l_max;
         p0 += gridDim.y * (step * kGroups)) {
      int32_t tk[kGroups];
      float ol[kGroups];
#pragma unroll
      for (int u = 0; u < kGroups; ++u) {
        const int64_t p = p0 + u * step;
        if constexpr (kSelect) {
          tk[u] = p < n ? arena_tokens[off + p] : 0;
          ol[u] = p < n ? arena_old[off + p] : 0.0f;
        } else {
          tk[u] = 0;
          ol[u] = 0.0f;
          if (p < n) {
            tk[u] = arena_tokens[off + p];
            ol[u] = arena_old[off + p];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kGroups; ++u) {
        const int64_t p = p0 + u * step;
        if (kGroups > 1 && p >= l_max) continue;
        tok_row[p] = tk[u];
        old_row[p] = ol[u];
        seq_row[p] = p < n ? (int32_t)j : -1;
      }
    }
  }
}

// Blocks (j, y): row j, which only its own draw decides.  One more column sums
// the lengths of all draws.
template <bool kRanks, bool kVec>
__global__ void __launch_bounds__(kFuseThreads) sample_padded_kernel(DrawParams p, Ranks ranks,
                                                                     DrawTable t) {
  __shared__ int64_t off_s[kRanks ? kLdsGranules : 1];
  __shared__ int64_t lds[kFuseThreads / 64];
  if (blockIdx.x == 0 && blockIdx.y != 0) return;
  View v{};
  if constexpr (kRanks) v = view_ranks<kFuseThreads>(ranks, off_s, lds);
  const DrawSet d = draw_set(p, v);
  if (blockIdx.x == 0) {
    int64_t sum = 0;
    for (int64_t j = threadIdx.x; j < p.n_draw; j += kFuseThreads)
      sum += stream_len(p, t.length[phys_row(draw_slot<kRanks>(p, d, v, j), p.head, p.cap)]);
    int64_t total;
    block_exclusive_scan<kFuseThreads>(sum, &total, lds);
    if (threadIdx.x == 0) {
      *t.n_tokens = total;
      t.cu_seqlens[0] = 0;
    }
    return;
  }
  const int64_t j = (int64_t)blockIdx.x - 1;
  const int64_t slot = draw_slot<kRanks>(p, d, v, j);
  const int64_t r = phys_row(slot, p.head, p.cap);
  const int64_t len = t.length[r], off = t.arena_off[r];
  if (blockIdx.y == 0 && threadIdx.x == 0) {
    write_draw(p, t, j, slot, r, len);
    t.cu_seqlens[j + 1] = (int32_t)((j + 1) * p.l_max);
  }
  fill_row<kVec, kVec ? kRowVecs : kRowSingles, kRanks>(j, p.l_max, stream_len(p, len), off,
                                                        t.arena_tokens, t.arena_old, t.tokens,
                                                        t.old_logp, t.seq);
}

// ---- draws, then the gather -------------------------------------------------

// Up to kDrawThreads draws: one block, one draw per thread, block scan of the
// lengths -> cu_seqlens, n_tokens.
template <bool kRanks>
__global__ void __launch_bounds__(kDrawThreads) draw_kernel(DrawParams p, Ranks ranks, DrawTable t,
                                                            int64_t* __restrict__ stream_total) {
  __shared__ int64_t off_s[kRanks ? kLdsGranules : 1];
  __shared__ int64_t lds[kDrawThreads / 64];
  View rv{};
  if constexpr (kRanks) rv = view_ranks<kDrawThreads>(ranks, off_s, lds);
  const DrawSet d = draw_set(p, rv);
  const int64_t j = threadIdx.x;
  const int64_t v = j < p.n_draw ? draw_one<kRanks>(p, d, rv, t, j) : 0;
  int64_t total;
  const int64_t ex = block_exclusive_scan<kDrawThreads>(v, &total, lds);
  if (j == 0) t.cu_seqlens[0] = 0;
  if (j < p.n_draw)
    t.cu_seqlens[j + 1] = (int32_t)(p.layout == RB_LAYOUT_PACKED ? ex + v : (j + 1) * p.l_max);
  if (j == 0) write_totals(p, total, t.n_tokens, stream_total);
}

// More draws: blocks of kRowThreads draws write the per-draw outputs and
// their block sums; one block scans the sums; then each block writes its
// cu_seqlens.  Many blocks keep the scattered record reads spread over the
// chip.
template <bool kRanks>
__global__ void __launch_bounds__(kRowThreads) draw_rows_kernel(DrawParams p, Ranks ranks,
                                                                DrawTable t,
                                                                int64_t* __restrict__ blk_sum) {
  __shared__ int64_t off_s[kRanks ? kLdsGranules : 1];
  __shared__ int64_t lds[kRowThreads / 64];
  View rv{};
  if constexpr (kRanks) rv = view_ranks<kRowThreads>(ranks, off_s, lds);
  const DrawSet d = draw_set(p, rv);
  const int64_t j = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
  const int64_t v = j < p.n_draw ? draw_one<kRanks>(p, d, rv, t, j) : 0;
  int64_t total;
  block_exclusive_scan<kRowThreads>(v, &total, lds);
  if (threadIdx.x == 0) blk_sum[blockIdx.x] = total;
}

__global__ void __launch_bounds__(1024) draw_scan_kernel(DrawParams p,
                                                         const int64_t* __restrict__ blk_sum,
                                                         int64_t* __restrict__ blk_off, int64_t nb,
                                                         int64_t* __restrict__ n_tokens,
                                                         int64_t* __restrict__ stream_total) {
  __shared__ int64_t lds[1024 / 64];
  int64_t carry = 0;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t v = i < nb ? blk_sum[i] : 0;
    int64_t total;
    const int64_t ex = block_exclusive_scan<1024>(v, &total, lds);
    if (i < nb) blk_off[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) write_totals(p, carry, n_tokens, stream_total);
}

__global__ void __launch_bounds__(kRowThreads) draw_cu_kernel(
    DrawParams p, const int32_t* __restrict__ out_len, const int64_t* __restrict__ blk_off,
    int32_t* __restrict__ cu_seqlens) {
  __shared__ int64_t lds[kRowThreads / 64];
  const int64_t j = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
  const int64_t v = j < p.n_draw ? (int64_t)out_len[j] : 0;
  int64_t total;
  const int64_t ex = block_exclusive_scan<kRowThreads>(v, &total, lds);
  if (j == 0) cu_seqlens[0] = 0;
  if (j < p.n_draw)
    cu_seqlens[j + 1] = (int32_t)(p.layout == RB_LAYOUT_PACKED ? blk_off[blockIdx.x] + ex + v
                                                               : (j + 1) * p.l_max);
}

// Block (j, y) copies the tokens of draw j that fall in the window
// [token_begin, token_begin + max_tokens) of the packed stream, rows y
// splitting long sequences; every block also takes its share of the window
// positions past the end of the stream, which are padded.
__global__ void __launch_bounds__(256) gather_packed_kernel(
    int64_t head, int64_t cap, int64_t token_begin, int64_t max_tokens,
    const int64_t* __restrict__ stream_total, const int32_t* __restrict__ cu_seqlens,
    const int32_t* __restrict__ idx, const int64_t* __restrict__ arena_off,
    const int32_t* __restrict__ arena_tokens, const float* __restrict__ arena_old,
    int32_t* __restrict__ tokens, float* __restrict__ old_logp, int32_t* __restrict__ seq) {
  const int64_t win_end = token_begin + max_tokens;
  const int64_t total = *stream_total;
  const int64_t n_blk = (int64_t)gridDim.x * gridDim.y;
  const int64_t blk = (int64_t)blockIdx.x * gridDim.y + blockIdx.y;
  for (int64_t pos = (total > token_begin ? total : token_begin) + blk * 256 + threadIdx.x;
       pos < win_end; pos += n_blk * 256) {
    const int64_t t = pos - token_begin;
    tokens[t] = 0;
    old_logp[t] = 0.0f;
    seq[t] = -1;
  }
  const int64_t j = blockIdx.x;
  const int64_t c0 = cu_seqlens[j], c1 = cu_seqlens[j + 1];
  const int64_t lo = c0 > token_begin ? c0 : token_begin;
  const int64_t hi = c1 < win_end ? c1 : win_end;
  if (lo >= hi) return;
  const int64_t src = arena_off[phys_row(idx[j], head, cap)] - c0;  // + stream position
  for (int64_t pos = lo + (int64_t)blockIdx.y * 256 + threadIdx.x; pos < hi;
       pos += (int64_t)gridDim.y * 256) {
    const int64_t t = pos - token_begin;
    tokens[t] = arena_tokens[src + pos];
    old_logp[t] = arena_old[src + pos];
    seq[t] = (int32_t)j;
  }
}

// Padded rows of draws already made.
template <bool kVec>
__global__ void __launch_bounds__(kFuseThreads) gather_padded_kernel(
    int64_t l_max, int64_t head, int64_t cap, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ len, const int64_t* __restrict__ arena_off,
    const int32_t* __restrict__ arena_tokens, const float* __restrict__ arena_old,
    int32_t* __restrict__ tokens, float* __restrict__ old_logp, int32_t* __restrict__ seq) {
  const int64_t j = blockIdx.x;
  const int64_t n = len[j] < l_max ? len[j] : l_max;
  fill_row<kVec, 1, false>(j, l_max, n, arena_off[phys_row(idx[j], head, cap)], arena_tokens,
                           arena_old, tokens, old_logp, seq);
}

// Workspace of a table of `capacity` rows.  Its size is part of the contract of
// rb_sample_gather_noalloc (which tables its static scratch holds), so it
// keeps room for a 4-byte slot list and two 4-byte counts per granule: the
// masks take the list's place.
struct SampleWs {
  uint64_t* mark;     // [2][nb * kWords]: marked slots, ties
  int64_t* meta;      // total of the ranks, length of the stream, ties to take
  uint64_t* keys;     // [capacity]
  int64_t *counts, *offsets;  // [nb]
  SelState* top;
  uint32_t *top_hist, *cand_cnt;
  uint64_t* cand;     // [capacity]
  int64_t *blk_sum, *blk_off;
  size_t bytes;
};

SampleWs carve_sample(void* base, int64_t capacity) {
  const int64_t nb = rbp::ceil_div(capacity, kGranule);
  rbp::WsCarver c(base);
  SampleWs w;
  c.take<int32_t>(nb);
  c.take<int32_t>(nb);
  // two sets of masks, 2 * nb * kWords * 8 <= capacity / 4 + 256 bytes: within
  // 4 * capacity rounded up to 256
  w.mark = reinterpret_cast<uint64_t*>(c.take<int32_t>(capacity));
  w.meta = c.take<int64_t>(4);
  w.keys = c.take<uint64_t>(capacity);
  w.counts = c.take<int64_t>(nb);
  w.offsets = c.take<int64_t>(nb);
  w.top = c.take<SelState>(1);
  w.top_hist = c.take<uint32_t>(kKeyBlocks * 256);
  w.cand_cnt = c.take<uint32_t>(kKeyBlocks);
  w.cand = c.take<uint64_t>(capacity);
  w.blk_sum = c.take<int64_t>(kMaxRowBlocks);
  w.blk_off = c.take<int64_t>(kMaxRowBlocks);
  w.bytes = rbp::align_up(c.used, 256);
  return w;
}

}  // namespace

size_t rbp::sample_gather_ws(int64_t capacity) {
  return carve_sample(nullptr, capacity < 1 ? 1 : capacity).bytes;
}

namespace {

// Everything rb_sample_gather does after clearing the error text: argument
// checks, then the device pipeline with `ws` as its workspace.
int sample_gather(const rb_records* rec, const rb_sample_cfg* cfg, const rb_batch* out, void* ws,
                  size_t ws_bytes, void* stream) {
  RBP_REQUIRE(rec && cfg && out, RBP_EINVAL, "rb_sample_gather: null struct pointer");
  RBP_REQUIRE(rec->capacity >= 1 && rec->n_live >= 1 && rec->n_live <= rec->capacity,
              RBP_EINVAL, "rb_sample_gather: need 1 <= n_live <= capacity (got %lld, %lld)",
              (long long)rec->n_live, (long long)rec->capacity);
  RBP_REQUIRE(rec->capacity <= INT32_MAX, RBP_EINVAL,
              "rb_sample_gather: capacity above 2^31-1");
  RBP_REQUIRE(rec->head >= 0 && rec->head < rec->capacity, RBP_EINVAL,
              "rb_sample_gather: head outside [0, capacity)");
  RBP_REQUIRE(rec->arena_off && rec->length && rec->reward && rec->advantage &&
                  rec->version && rec->arena_tokens && rec->arena_old_logp,
              RBP_EINVAL, "rb_sample_gather: null record array");
  RBP_REQUIRE(cfg->mode >= RB_UNIFORM && cfg->mode <= RB_UNUSED_FIRST, RBP_EINVAL,
              "rb_sample_gather: unknown mode %d", cfg->mode);
  const bool no_replace = cfg->mode == RB_NO_REPLACE || cfg->mode == RB_UNUSED_FIRST;
  RBP_REQUIRE(!no_replace || cfg->n_draw <= rec->n_live, RBP_EINVAL,
              "rb_sample_gather: %lld draws without replacement from %lld records",
              (long long)cfg->n_draw, (long long)rec->n_live);
  RBP_REQUIRE(cfg->mode != RB_UNUSED_FIRST || rec->use_count != nullptr, RBP_EINVAL,
              "rb_sample_gather: RB_UNUSED_FIRST needs use_count");
  RBP_REQUIRE(cfg->layout == RB_LAYOUT_PACKED || cfg->layout == RB_LAYOUT_PADDED, RBP_EINVAL,
              "rb_sample_gather: unknown layout %d", cfg->layout);
  RBP_REQUIRE(cfg->n_draw >= 1 && cfg->n_draw <= (1 << 20), RBP_EINVAL,
              "rb_sample_gather: n_draw %lld outside [1, 2^20]", (long long)cfg->n_draw);
  RBP_REQUIRE(cfg->p_pos_q32 <= (1ull << 32), RBP_EINVAL,
              "rb_sample_gather: p_pos_q32 above 2^32");
  RBP_REQUIRE(cfg->n_fresh >= 0 && cfg->n_pos_keep >= 0, RBP_EINVAL,
              "rb_sample_gather: negative n_fresh / n_pos_keep");
  if (cfg->layout == RB_LAYOUT_PACKED) {
    RBP_REQUIRE(cfg->max_tokens >= 1 && cfg->token_begin >= 0, RBP_EINVAL,
                "rb_sample_gather: packed layout needs max_tokens >= 1, token_begin >= 0");
  } else {
    RBP_REQUIRE(cfg->l_max >= 1 && cfg->n_draw * cfg->l_max <= INT32_MAX, RBP_EINVAL,
                "rb_sample_gather: padded layout needs l_max >= 1 and n_draw * l_max < 2^31");
  }
  RBP_REQUIRE(out->idx && out->adv && out->len && out->age && out->cu_seqlens && out->tokens &&
                  out->old_logp && out->seq_of_token && out->n_tokens,
              RBP_EINVAL, "rb_sample_gather: null output array");
  const size_t need = rbp::sample_gather_ws(rec->capacity);
  RBP_REQUIRE(ws && ws_bytes >= need, RBP_EWORKSPACE,
              "rb_sample_gather: workspace needs %zu bytes, got %zu", need, ws_bytes);

  hipStream_t s = rbp::as_stream(stream);
  const SampleWs w = carve_sample(ws, rec->capacity);

  DrawParams p{};
  p.mode = cfg->mode;
  p.layout = cfg->layout;
  p.seed = cfg->seed;
  p.step = cfg->step;
  p.p_q32 = cfg->p_pos_q32;
  p.n_draw = cfg->n_draw;
  p.n_live = rec->n_live;
  p.head = rec->head;
  p.cap = rec->capacity;
  p.first_fresh = rec->n_live - cfg->n_fresh;
  if (p.first_fresh < 0) p.first_fresh = 0;
  p.n_pos_keep = cfg->n_pos_keep;
  p.cur_version = cfg->cur_version;
  p.max_tokens = cfg->max_tokens;
  p.token_begin = cfg->token_begin;
  p.l_max = cfg->l_max;

  Ranks ranks{};
  if (no_replace) {
    const int64_t n = rec->n_live;
    int64_t kb = rbp::ceil_div(n, kKeyThreads);
    if (kb > kKeyBlocks) kb = kKeyBlocks;
    hipLaunchKernelGGL(slot_key_kernel, dim3(kb), dim3(kKeyThreads), 0, s, cfg->seed, cfg->step,
                       n, rec->head, rec->capacity,
                       cfg->mode == RB_UNUSED_FIRST ? rec->use_count : nullptr, w.keys,
                       w.top_hist);
    hipLaunchKernelGGL(select_cand_kernel, dim3(kb), dim3(kKeyThreads), 0, s, w.keys, n,
                       w.top_hist, cfg->n_draw, w.top, w.cand, w.cand_cnt);
    ranks.nb = (int32_t)rbp::ceil_div(n, kGranule);
    uint64_t* tie = w.mark + (int64_t)ranks.nb * kWords;
    const unsigned blocks = ranks.nb < 256 ? ranks.nb : 256;
    hipLaunchKernelGGL(select_rest_kernel, dim3(blocks), dim3(kRestThreads), 0, s, w.keys, n, w.top,
                       w.cand, w.cand_cnt, (int32_t)kb, ranks.nb, w.mark, tie, w.counts,
                       w.meta + 2);
    ranks.tie = tie;
    ranks.need = w.meta + 2;
  } else if (cfg->mode != RB_UNIFORM) {
    // positives over all live slots (mixture) or over the non-fresh ones (retention)
    const int64_t n_range = cfg->mode == RB_POS_MIX ? rec->n_live : p.first_fresh;
    ranks.nb = (int32_t)rbp::ceil_div(n_range > 0 ? n_range : 1, kGranule);
    hipLaunchKernelGGL(pos_mask_kernel, dim3(ranks.nb), dim3(kMaskThreads), 0, s, rec->reward,
                       rec->head, rec->capacity, n_range, w.mark, w.counts);
  }
  ranks.mark = w.mark;
  ranks.counts = w.counts;
  if (ranks.nb > kLdsGranules) {
    hipLaunchKernelGGL(rank_scan_kernel, dim3(1), dim3(1024), 0, s, w.counts, w.offsets,
                       (int64_t)ranks.nb, w.meta);
    ranks.offsets = w.offsets;
    ranks.total = w.meta;
  }
  const DrawTable t{rec->length,     rec->advantage,      rec->version, rec->arena_off,
                    rec->arena_tokens, rec->arena_old_logp, out->idx,     out->adv,
                    out->len,        out->age,            out->cu_seqlens, out->tokens,
                    out->old_logp,   out->seq_of_token,   out->n_tokens};
  const bool packed = cfg->layout == RB_LAYOUT_PACKED;
  const bool vec = cfg->l_max % 4 == 0 &&
                   ((reinterpret_cast<uintptr_t>(out->tokens) |
                     reinterpret_cast<uintptr_t>(out->old_logp) |
                     reinterpret_cast<uintptr_t>(out->seq_of_token)) & 15) == 0;
  // Draw and gather in one launch while every block can redo the draws it
  // needs at little cost.  Padded, that is one draw, and one block sums all of
  // them (padded_one_launch); packed, it is all of them (packed_route).
  const auto route = packed ? rbp::rules::packed_route(cfg->n_draw, cfg->max_tokens, ranks.nb > 0)
                            : rbp::rules::PackedRoute{0, 0, 0};
  if (route.blocks > 0) {
    constexpr int kS = rbp::rules::kPackedSmall, kL = rbp::rules::kPackedLarge;
    const bool rk = ranks.nb > 0;
    const auto kernel =
        route.threads == kS
            ? (rk ? sample_packed_kernel<true, kS, 1> : sample_packed_kernel<false, kS, 1>)
            : (route.positions == 1
                   ? (rk ? sample_packed_kernel<true, kL, 1> : sample_packed_kernel<false, kL, 1>)
                   : (rk ? sample_packed_kernel<true, kL, 2> : sample_packed_kernel<false, kL, 2>));
    hipLaunchKernelGGL(kernel, dim3((unsigned)route.blocks), dim3(route.threads), 0, s, p, ranks,
                       t);
    RBP_CHECK_LAUNCH("rb_sample_gather");
    return RBP_OK;
  }
  if (!packed && rbp::rules::padded_one_launch(cfg->n_draw, cfg->l_max, ranks.nb)) {
    const auto kernel = ranks.nb > 0
                            ? (vec ? sample_padded_kernel<true, true>
                                   : sample_padded_kernel<true, false>)
                            : (vec ? sample_padded_kernel<false, true>
                                   : sample_padded_kernel<false, false>);
    // blocks per row: as many as its passes, but no more in all than run at
    // once (5 per compute unit): each redoes the draw, and a second round of
    // them cost more than the longer rows (662 uniform draws of 2886 positions
    // 27.9 us in 12 blocks each, 13.5 in one)
    int64_t by = rbp::ceil_div(cfg->l_max, 256 * (vec ? 4 * kRowVecs : kRowSingles));
    if (by > 1280 / cfg->n_draw) by = 1280 / cfg->n_draw;
    hipLaunchKernelGGL(kernel, dim3((unsigned)cfg->n_draw + 1, (unsigned)by),
                       dim3(kFuseThreads), 0, s, p, ranks, t);
    RBP_CHECK_LAUNCH("rb_sample_gather");
    return RBP_OK;
  }
  if (cfg->n_draw <= kDrawThreads) {
    hipLaunchKernelGGL(ranks.nb > 0 ? draw_kernel<true> : draw_kernel<false>, dim3(1),
                       dim3(kDrawThreads), 0, s, p, ranks, t, w.meta + 1);
  } else {
    const int64_t nb = rbp::ceil_div(cfg->n_draw, kRowThreads);
    hipLaunchKernelGGL(ranks.nb > 0 ? draw_rows_kernel<true> : draw_rows_kernel<false>, dim3(nb),
                       dim3(kRowThreads), 0, s, p, ranks, t, w.blk_sum);
    hipLaunchKernelGGL(draw_scan_kernel, dim3(1), dim3(1024), 0, s, p, w.blk_sum, w.blk_off, nb,
                       out->n_tokens, w.meta + 1);
    hipLaunchKernelGGL(draw_cu_kernel, dim3(nb), dim3(kRowThreads), 0, s, p, out->len, w.blk_off,
                       out->cu_seqlens);
  }
  if (packed) {
    // about 256 window positions per block
    int64_t gy = rbp::ceil_div(cfg->max_tokens, cfg->n_draw * 256);
    if (gy > 64) gy = 64;
    hipLaunchKernelGGL(gather_packed_kernel, dim3(cfg->n_draw, gy), dim3(256), 0, s,
                       rec->head, rec->capacity, cfg->token_begin, cfg->max_tokens, w.meta + 1,
                       out->cu_seqlens, out->idx, rec->arena_off, rec->arena_tokens,
                       rec->arena_old_logp, out->tokens, out->old_logp, out->seq_of_token);
  } else {
    int64_t by = rbp::ceil_div(cfg->l_max, vec ? 1024 : 256);
    if (by > 64) by = 64;
    hipLaunchKernelGGL(vec ? gather_padded_kernel<true> : gather_padded_kernel<false>,
                       dim3(cfg->n_draw, by), dim3(kFuseThreads), 0, s, cfg->l_max, rec->head,
                       rec->capacity, out->idx, out->len, rec->arena_off, rec->arena_tokens,
                       rec->arena_old_logp, out->tokens, out->old_logp, out->seq_of_token);
  }
  RBP_CHECK_LAUNCH("rb_sample_gather");
  return RBP_OK;
}

// Workspace of rb_sample_gather_noalloc: one array per device, held from
// module load until the process ends.  In host code `scratch` names a
// host-side stand-in; the device address comes from hipGetSymbolAddress.
constexpr size_t kScratchBytes = size_t(32) << 20;
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_addr[kMaxDevices];
std::mutex g_scratch_lock;

// The current device's address of `scratch`, resolved on the first call on
// that device (with the device current) and kept.
int scratch_addr(void** addr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  RBP_REQUIRE(e == hipSuccess, RBP_EHIP, "rb_sample_gather_noalloc: hipGetDevice: %s",
              hipGetErrorString(e));
  RBP_REQUIRE(dev >= 0 && dev < kMaxDevices, RBP_EUNSUPPORTED,
              "rb_sample_gather_noalloc: device %d beyond the %d the library tracks", dev,
              kMaxDevices);
  void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    std::lock_guard<std::mutex> g(g_scratch_lock);
    p = g_scratch_addr[dev].load(std::memory_order_relaxed);
    if (p == nullptr) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      RBP_REQUIRE(e == hipSuccess && p != nullptr, RBP_EHIP,
                  "rb_sample_gather_noalloc: hipGetSymbolAddress(scratch) on device %d: %s",
                  dev, hipGetErrorString(e));
      g_scratch_addr[dev].store(p, std::memory_order_release);
    }
  }
  *addr = p;
  return RBP_OK;
}

}  // namespace

extern "C" int rb_sample_gather(const rb_records* rec, const rb_sample_cfg* cfg,
                                const rb_batch* out, void* ws, size_t ws_bytes,
                                void* stream) {
  rbp::clear_error();
  return sample_gather(rec, cfg, out, ws, ws_bytes, stream);
}

extern "C" int rb_sample_gather_noalloc(const rb_records* rec, const rb_sample_cfg* cfg,
                                        const rb_batch* out, void* stream) {
  rbp::clear_error();
  RBP_REQUIRE(rec, RBP_EINVAL, "rb_sample_gather_noalloc: null record table");
  RBP_REQUIRE(rec->capacity >= 1 && rec->capacity <= INT32_MAX, RBP_EINVAL,
              "rb_sample_gather_noalloc: capacity %lld outside [1, 2^31-1]",
              (long long)rec->capacity);
  const size_t need = rbp::sample_gather_ws(rec->capacity);
  RBP_REQUIRE(need <= kScratchBytes, RBP_EWORKSPACE,
              "rb_sample_gather_noalloc: a record table of capacity %lld needs %zu bytes of "
              "workspace, more than the %zu-byte static scratch (use rb_sample_gather with a "
              "caller workspace)",
              (long long)rec->capacity, need, kScratchBytes);
  void* ws = nullptr;
  const int st = scratch_addr(&ws);
  if (st != RBP_OK) return st;
  return sample_gather(rec, cfg, out, ws, kScratchBytes, stream);
}
