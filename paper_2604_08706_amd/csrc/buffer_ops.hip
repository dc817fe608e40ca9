// Buffer maintenance: FIFO insertion of generated groups (rb_push),
// per-record usage bookkeeping (rb_note_use) and the histograms of the buffer
// statistics (rb_hist_accumulate).
//
// Paper: the buffer holds the N most recent rollouts; a push into a full
// buffer evicts the oldest one and sampling never removes (App. B
// "BufferStructure"); advantages are computed once, when a group is generated
// (App. D.2).  Steps-since-last-use (App. D.3, "Metrics"): a rollout's first
// sample is "new", a later one gets the gradient steps since its previous
// sample, 0 for repeats inside one batch.  Sec. 3.2 reports the distributions
// of off-policiness (a sample's age), replay ratio (uses of a rollout over the
// run) and steps since last use.
//
// The record table is a ring: logical slot s is physical row (head + s) %
// capacity, and row r owns a fixed arena stretch of slot_tokens tokens, so an
// inserted record always overwrites the storage of the record it evicts.
// Everything here is integer work or a copy, except the advantage (fp32, the
// arithmetic of rb_group_advantage).

#include "group_advantage.h"
#include "launch_rules.h"
#include "rbp_internal.h"

namespace {

__device__ __forceinline__ int64_t ring_row(int64_t base, int64_t i, int64_t cap) {
  const int64_t r = base + i;
  return r >= cap ? r - cap : r;
}

constexpr int kHistMaxBins = 4096;
using rbp::rules::kPushLoads;
using rbp::rules::kPushThreads;
using rbp::rules::kPushTokens;

struct PushRing {
  int64_t base, cap, slot_tokens;  // base: the first new record's row
  int64_t* off;
  int32_t* len;
  float *reward, *advantage;
  int32_t *version, *uses;
  int64_t* last;
  int32_t* tokens;
  float* old_logp;
  int64_t* hist;
  int32_t n_bins;
  int64_t first_evict;  // new records from here on overwrite a live one
};

// One launch for a whole push (four launches of 2 to 7 us, each waiting for
// the one before, took 29.5 us for 1024 records of about 900 tokens; bound by
// launches and load latency, the bytes are worth 3 us).  Its parts are
// independent of each other; the ones with the longest chains come first:
//   group_blocks blocks: the advantages of 256 groups each, straight into the
//     ring rows;
//   field_blocks blocks: the fields of 256 records each, after the evicted
//     records' use counts -- their replay ratios (Sec. 3.2) -- are counted in
//     LDS and added to the histogram bin by bin (an atomic per record on a
//     dozen hot bins took longer than the copy);
//   the others: one column per record, the rows of the grid splitting long
//     ones, copy tokens and behaviour log-probs into the records' arena
//     stretches (at most slot_tokens of them).
__global__ void __launch_bounds__(kPushThreads) push_kernel(
    PushRing ring, int32_t n_new, int32_t group_blocks, int32_t field_blocks, int32_t n_groups,
    const int32_t* __restrict__ group_off, const int32_t* __restrict__ length,
    const int64_t* __restrict__ src_off, const float* __restrict__ reward, int32_t version,
    const int32_t* __restrict__ tokens, const float* __restrict__ old_logp, int32_t ddof,
    float eps) {
  __shared__ union {
    float r[rbp::kAdvStage];
    uint32_t h[kHistMaxBins];
  } lds;
  int32_t b = (int32_t)blockIdx.x;
  if (b < group_blocks) {
    if (blockIdx.y != 0) return;
    const int32_t g0 = b * kPushThreads;
    const int32_t g1 = g0 + kPushThreads < n_groups ? g0 + kPushThreads : n_groups;
    const int32_t g = g0 + (int32_t)threadIdx.x;
    const int32_t lo = group_off[g0], n = group_off[g1] - lo;
    auto out = [&](int32_t k, float a) {
      ring.advantage[ring_row(ring.base, k, ring.cap)] = a;
    };
    if (n > rbp::kAdvStage) {
      if (g < g1)
        rbp::group_advantage(reward, group_off[g], group_off[g + 1], ddof, eps, out);
      return;
    }
    for (int32_t k = threadIdx.x; k < n; k += kPushThreads) lds.r[k] = reward[lo + k];
    __syncthreads();
    if (g < g1)
      rbp::group_advantage(lds.r, group_off[g] - lo, group_off[g + 1] - lo, ddof, eps,
                           [&](int32_t k, float a) { out(lo + k, a); });
    return;
  }
  b -= group_blocks;
  if (b < field_blocks) {
    if (blockIdx.y != 0) return;
    const int32_t i = b * kPushThreads + (int32_t)threadIdx.x;
    const int64_t r = ring_row(ring.base, i, ring.cap);
    if (ring.hist != nullptr && ring.first_evict < n_new) {
      for (int32_t k = threadIdx.x; k < ring.n_bins; k += kPushThreads) lds.h[k] = 0u;
      __syncthreads();
      if (i < n_new && i >= ring.first_evict) {
        const int32_t u = ring.uses[r];
        atomicAdd(&lds.h[u < 0 ? 0 : (u > ring.n_bins - 1 ? ring.n_bins - 1 : u)], 1u);
      }
      __syncthreads();
      for (int32_t k = threadIdx.x; k < ring.n_bins; k += kPushThreads)
        if (lds.h[k] != 0u)
          atomicAdd(reinterpret_cast<unsigned long long*>(ring.hist + k),
                    (unsigned long long)lds.h[k]);
    }
    if (i >= n_new) return;
    const int32_t len = length[i];
    ring.off[r] = r * ring.slot_tokens;
    ring.len[r] = (int64_t)len < ring.slot_tokens ? len : (int32_t)ring.slot_tokens;
    ring.reward[r] = reward[i];
    ring.version[r] = version;
    if (ring.uses != nullptr) ring.uses[r] = 0;
    if (ring.last != nullptr) ring.last[r] = -1;
    return;
  }
  b -= field_blocks;
  const int32_t rec_blocks = (int32_t)gridDim.x - group_blocks - field_blocks;
  for (int64_t i = b; i < n_new; i += rec_blocks) {
    const int64_t r = ring_row(ring.base, i, ring.cap);
    const int32_t len = length[i];
    const int64_t n = (int64_t)len < ring.slot_tokens ? len : ring.slot_tokens;
    const int64_t src = src_off[i], dst = r * ring.slot_tokens;
    for (int64_t p0 = (int64_t)blockIdx.y * kPushTokens; p0 < n;
         p0 += (int64_t)gridDim.y * kPushTokens) {
      int32_t tk[kPushLoads];
      float ol[kPushLoads];
#pragma unroll
      for (int k = 0; k < kPushLoads; ++k) {  // all loads in flight before the first store
        const int64_t p = p0 + k * kPushThreads + threadIdx.x;
        tk[k] = p < n ? tokens[src + p] : 0;
        ol[k] = p < n ? old_logp[src + p] : 0.0f;
      }
#pragma unroll
      for (int k = 0; k < kPushLoads; ++k) {
        const int64_t p = p0 + k * kPushThreads + threadIdx.x;
        if (p < n) {
          ring.tokens[dst + p] = tk[k];
          ring.old_logp[dst + p] = ol[k];
        }
      }
    }
  }
}

// ---- usage bookkeeping ------------------------------------------------------

__device__ __forceinline__ int64_t drawn_row(const int32_t* __restrict__ idx, int64_t j,
                                             int64_t head, int64_t cap) {
  return ring_row(head, idx[j], cap);
}

__global__ void __launch_bounds__(256) use_reset_kernel(const int32_t* __restrict__ idx,
                                                        int64_t n, int64_t head, int64_t cap,
                                                        int32_t* __restrict__ first) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256)
    first[drawn_row(idx, j, head, cap)] = INT32_MAX;
}

// first[row] = smallest draw index of the batch that took the row
__global__ void __launch_bounds__(256) use_first_kernel(const int32_t* __restrict__ idx,
                                                        int64_t n, int64_t head, int64_t cap,
                                                        int32_t* __restrict__ first) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256)
    atomicMin(&first[drawn_row(idx, j, head, cap)], (int32_t)j);
}

__global__ void __launch_bounds__(256) use_since_kernel(const int32_t* __restrict__ idx,
                                                        int64_t n, int64_t head, int64_t cap,
                                                        int64_t step,
                                                        const int32_t* __restrict__ first,
                                                        const int64_t* __restrict__ last,
                                                        int32_t* __restrict__ since) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * 256) {
    const int64_t r = drawn_row(idx, j, head, cap);
    const int64_t l = last[r];
    since[j] = first[r] < j ? 0 : (l < 0 ? -1 : (int32_t)(step - l));
  }
}

// use_count += draws of the row (integer atomics: the sum is order-free);
// the row's first draw stores the step.
__global__ void __launch_bounds__(256) use_update_kernel(const int32_t* __restrict__ idx,
                                                         int64_t n, int64_t head, int64_t cap,
                                                         int64_t step,
                                                         const int32_t* __restrict__ first,
                                                         int32_t* __restrict__ uses,
                                                         int64_t* __restrict__ last) {
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * 256) {
    const int64_t r = drawn_row(idx, j, head, cap);
    atomicAdd(&uses[r], 1);
    if (first[r] == j) last[r] = step;
  }
}

// Up to kUseThreads draws: one block, with the drawn rows in a hash table in
// LDS (twice as many places as draws, so a probe ends) instead of the table of
// first draws: one launch in place of the four above, each of which waits for
// the one before (512 draws, calls back to back in a graph: 3.0 us each against
// 8.1; 1024 4.5 / 8.7).  Which place a row gets depends on the order of the
// insertions, its first draw and its number of draws do not.
constexpr int kUseThreads = 1024;
constexpr int kUsePlaces = 2 * kUseThreads;

__global__ void __launch_bounds__(kUseThreads) use_small_kernel(
    const int32_t* __restrict__ idx, int32_t n, int64_t head, int64_t cap, int64_t step,
    int32_t* __restrict__ uses, int64_t* __restrict__ last, int32_t* __restrict__ since) {
  __shared__ int32_t key[kUsePlaces], first[kUsePlaces], draws[kUsePlaces];
  const int32_t j = (int32_t)threadIdx.x;
  for (int32_t k = j; k < kUsePlaces; k += kUseThreads) {
    key[k] = -1;  // slots are not negative
    first[k] = INT32_MAX;
    draws[k] = 0;
  }
  const int32_t slot = j < n ? idx[j] : 0;
  const int64_t r = ring_row(head, slot, cap);
  const int64_t l = j < n ? last[r] : 0;
  const int32_t u = j < n ? uses[r] : 0;
  __syncthreads();
  int32_t at = (int32_t)(((uint32_t)slot * 2654435761u) >> 21);  // 11 bits: kUsePlaces
  if (j < n) {
    for (int32_t probe = 0; probe < kUsePlaces; ++probe) {
      const int32_t was = atomicCAS(&key[at], -1, slot);
      if (was == -1 || was == slot) break;
      at = (at + 1) & (kUsePlaces - 1);
    }
    atomicMin(&first[at], j);
    atomicAdd(&draws[at], 1);
  }
  __syncthreads();
  if (j >= n) return;
  const bool is_first = first[at] == j;
  if (since != nullptr) since[j] = !is_first ? 0 : (l < 0 ? -1 : (int32_t)(step - l));
  if (is_first) {
    uses[r] = u + draws[at];
    last[r] = step;
  }
}

// ---- statistics ------------------------------------------------------------

// Block histogram in LDS, then one integer atomic per non-empty bin.
__global__ void __launch_bounds__(256) hist_kernel(const int32_t* __restrict__ values, int64_t n,
                                                   int32_t lo, int32_t n_bins,
                                                   int64_t* __restrict__ hist) {
  __shared__ uint32_t h[kHistMaxBins];
  for (int b = threadIdx.x; b < n_bins; b += 256) h[b] = 0u;
  __syncthreads();
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
    int64_t b = (int64_t)values[j] - lo;
    b = b < 0 ? 0 : (b > n_bins - 1 ? n_bins - 1 : b);
    atomicAdd(&h[b], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < n_bins; b += 256)
    if (h[b] != 0u) atomicAdd(reinterpret_cast<unsigned long long*>(hist + b), (unsigned long long)h[b]);
}

}  // namespace

size_t rbp::note_use_ws(int64_t capacity) {
  return align_up(sizeof(int32_t) * (size_t)(capacity < 1 ? 1 : capacity), 256);
}

extern "C" int rb_push(rb_ring* ring, int32_t n_new, int32_t n_groups, const int32_t* group_off,
                       const int32_t* length, const int64_t* src_off, const float* reward,
                       int32_t version, const int32_t* tokens, const float* old_logp,
                       int32_t ddof, float eps, void* stream) {
  rbp::clear_error();
  RBP_REQUIRE(ring != nullptr, RBP_EINVAL, "rb_push: null ring");
  const int64_t cap = ring->capacity;
  RBP_REQUIRE(cap >= 1 && cap <= INT32_MAX, RBP_EINVAL, "rb_push: capacity outside [1, 2^31)");
  RBP_REQUIRE(ring->n_live >= 0 && ring->n_live <= cap, RBP_EINVAL,
              "rb_push: n_live outside [0, capacity]");
  RBP_REQUIRE(ring->head >= 0 && ring->head < cap, RBP_EINVAL, "rb_push: head outside [0, capacity)");
  RBP_REQUIRE(ring->slot_tokens >= 1, RBP_EINVAL, "rb_push: slot_tokens < 1");
  RBP_REQUIRE(n_new >= 1 && n_new <= cap, RBP_EINVAL, "rb_push: n_new %d outside [1, capacity]",
              n_new);
  RBP_REQUIRE(n_groups >= 1, RBP_EINVAL, "rb_push: n_groups < 1");
  RBP_REQUIRE(ddof == 0 || ddof == 1, RBP_EINVAL, "rb_push: ddof must be 0 or 1");
  RBP_REQUIRE(eps >= 0.0f, RBP_EINVAL, "rb_push: eps < 0");
  RBP_REQUIRE(ring->arena_off && ring->length && ring->reward && ring->advantage &&
                  ring->version && ring->arena_tokens && ring->arena_old_logp,
              RBP_EINVAL, "rb_push: null ring array");
  RBP_REQUIRE(group_off && length && src_off && reward && tokens && old_logp, RBP_EINVAL,
              "rb_push: null input array");
  RBP_REQUIRE(ring->replay_hist == nullptr ||
                  (ring->use_count != nullptr && ring->replay_bins >= 1 &&
                   ring->replay_bins <= kHistMaxBins),
              RBP_EINVAL, "rb_push: replay_hist needs use_count and 1 <= replay_bins <= %d",
              kHistMaxBins);
  hipStream_t s = rbp::as_stream(stream);
  // the first free row: just past the newest record
  int64_t base = ring->head + ring->n_live;
  if (base >= cap) base -= cap;
  const PushRing pr{base,
                    cap,
                    ring->slot_tokens,
                    ring->arena_off,
                    ring->length,
                    ring->reward,
                    ring->advantage,
                    ring->version,
                    ring->use_count,
                    ring->last_step,
                    ring->arena_tokens,
                    ring->arena_old_logp,
                    ring->replay_hist,
                    ring->replay_bins,
                    cap - ring->n_live};
  const int64_t by = rbp::rules::push_rows(n_new, ring->slot_tokens);
  // a launch holds 2^32 threads, 2^24 blocks: at most 2^21 blocks of records
  // beside the (at most 2^23) blocks of groups and of fields, which lie below
  // 2^24 together unless both counts are near 2^31
  const int32_t rec_blocks = n_new < (1 << 21) ? n_new : (1 << 21);
  const int32_t group_blocks = (int32_t)rbp::ceil_div(n_groups, kPushThreads);
  const int32_t field_blocks = (int32_t)rbp::ceil_div(n_new, kPushThreads);
  hipLaunchKernelGGL(push_kernel,
                     dim3((unsigned)(rec_blocks + group_blocks + field_blocks), (unsigned)by),
                     dim3(kPushThreads), 0, s, pr, n_new, group_blocks, field_blocks, n_groups,
                     group_off, length, src_off, reward, version, tokens, old_logp, ddof, eps);
  RBP_CHECK_LAUNCH("rb_push");
  // FIFO bookkeeping (host integers): records past the capacity evict the oldest
  const int64_t total = ring->n_live + n_new;
  const int64_t evicted = total > cap ? total - cap : 0;
  ring->head = (ring->head + evicted) % cap;
  ring->n_live = total - evicted;
  return RBP_OK;
}

extern "C" int rb_note_use(const int32_t* idx, int64_t n_draw, int64_t head, int64_t capacity,
                           int64_t step, int32_t* use_count, int64_t* last_step, int32_t* since,
                           void* ws, size_t ws_bytes, void* stream) {
  rbp::clear_error();
  RBP_REQUIRE(n_draw >= 0, RBP_EINVAL, "rb_note_use: n_draw < 0");
  RBP_REQUIRE(capacity >= 1 && capacity <= INT32_MAX && head >= 0 && head < capacity,
              RBP_EINVAL, "rb_note_use: need 1 <= capacity < 2^31 and 0 <= head < capacity");
  RBP_REQUIRE(step >= 0, RBP_EINVAL, "rb_note_use: step < 0");
  if (n_draw == 0) return RBP_OK;
  RBP_REQUIRE(idx && use_count && last_step, RBP_EINVAL, "rb_note_use: null pointer");
  const size_t need = rbp::note_use_ws(capacity);
  RBP_REQUIRE(ws && ws_bytes >= need, RBP_EWORKSPACE,
              "rb_note_use: workspace needs %zu bytes, got %zu", need, ws_bytes);
  hipStream_t s = rbp::as_stream(stream);
  if (n_draw <= kUseThreads) {
    hipLaunchKernelGGL(use_small_kernel, dim3(1), dim3(kUseThreads), 0, s, idx, (int32_t)n_draw,
                       head, capacity, step, use_count, last_step, since);
    RBP_CHECK_LAUNCH("rb_note_use");
    return RBP_OK;
  }
  int32_t* first = static_cast<int32_t*>(ws);
  int64_t blocks = rbp::ceil_div(n_draw, 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(use_reset_kernel, dim3(blocks), dim3(256), 0, s, idx, n_draw, head,
                     capacity, first);
  hipLaunchKernelGGL(use_first_kernel, dim3(blocks), dim3(256), 0, s, idx, n_draw, head,
                     capacity, first);
  if (since != nullptr)
    hipLaunchKernelGGL(use_since_kernel, dim3(blocks), dim3(256), 0, s, idx, n_draw, head,
                       capacity, step, first, last_step, since);
  hipLaunchKernelGGL(use_update_kernel, dim3(blocks), dim3(256), 0, s, idx, n_draw, head,
                     capacity, step, first, use_count, last_step);
  RBP_CHECK_LAUNCH("rb_note_use");
  return RBP_OK;
}

extern "C" int rb_hist_accumulate(const int32_t* values, int64_t n, int32_t lo, int32_t n_bins,
                                  int64_t* hist, void* stream) {
  rbp::clear_error();
  RBP_REQUIRE(n >= 0, RBP_EINVAL, "rb_hist_accumulate: n < 0");
  RBP_REQUIRE(n_bins >= 1 && n_bins <= kHistMaxBins, RBP_EINVAL,
              "rb_hist_accumulate: n_bins %d outside [1, %d]", n_bins, kHistMaxBins);
  if (n == 0) return RBP_OK;
  RBP_REQUIRE(values && hist, RBP_EINVAL, "rb_hist_accumulate: null pointer");
  int64_t blocks = rbp::ceil_div(n, 256 * 8);
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(hist_kernel, dim3(blocks), dim3(256), 0, rbp::as_stream(stream), values, n,
                     lo, n_bins, hist);
  RBP_CHECK_LAUNCH("rb_hist_accumulate");
  return RBP_OK;
}
