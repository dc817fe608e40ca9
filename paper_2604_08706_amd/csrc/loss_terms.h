// The clipped GRPO objective of one token (App. D.2) and the sums over tokens,
// shared by policy_loss_fwd_bwd and the single pass.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rbp {
namespace loss {

constexpr int kNumSums = 5;       // -sum w*l, sum rho, n clipped, n valid, sum l
constexpr int kMaxBlocks = 1024;  // rows of partial sums a workspace holds

// Loss terms of one token (a masked token, s < 0, contributes nothing).
struct TokenTerms {
  float g, wterm, rho, cut, valid, term;
};
__device__ __forceinline__ TokenTerms token_terms(float lp, float olp, int32_t s,
                                                  const float* __restrict__ adv,
                                                  const int32_t* __restrict__ seq_len,
                                                  float inv_nseq, float lo_b, float hi_b) {
  TokenTerms r{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (s < 0) return r;
  const float A = adv[s];
  const float w = inv_nseq / (float)seq_len[s];
  const float rho = expf(lp - olp);
  const float clipped = fminf(fmaxf(rho, lo_b), hi_b);
  const float term = fminf(rho * A, clipped * A);
  const bool cut = (A > 0.0f && rho > hi_b) || (A < 0.0f && rho < lo_b);
  r.g = cut ? 0.0f : -A * rho * w;
  r.wterm = term * w;
  r.rho = rho;
  r.cut = cut ? 1.0f : 0.0f;
  r.valid = 1.0f;
  r.term = term;
  return r;
}

// One wave: sum k of the partial rows, lane l taking rows l, l + 64, ... in
// order, then a fixed butterfly over the lanes (bitwise reproducible).
__device__ __forceinline__ float sum_partials(const float* __restrict__ partials, int nblocks,
                                              int k) {
  float v = 0.0f;
  for (int b = threadIdx.x & 63; b < nblocks; b += 64) v += partials[b * kNumSums + k];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Its addition to the caller's accumulators, by one lane.
__device__ __forceinline__ void add_sum(int k, float v, float* __restrict__ loss_accum,
                                        float* __restrict__ stats) {
  if (k == 0)
    loss_accum[0] += v;
  else
    stats[k - 1] += v;
}

}  // namespace loss
}  // namespace rbp
