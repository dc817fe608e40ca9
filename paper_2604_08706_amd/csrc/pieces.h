// Cutting the K range of a launch's last round.
//
// A persistent product runs its tiles in rounds of G workgroups; a last round
// of r < G tiles leaves G - r compute units idle for a whole tile (a 7B-head
// micro-batch of 1301 tokens has 84 dhidden tiles on 256 units, one of 256
// tokens has 14).  Its tiles are cut along K instead: every tile into p
// pieces of `steps` K steps, every workgroup running q pieces, so that the
// round takes q / p of a tile and r p / q workgroups (at most G).
//
// Tile i has u = p / q workgroups of its own, number a running its pieces
// a q .. a q + q - 1 back to back; the rem = p % q pieces left over go, tile
// after tile, to helper workgroups of q pieces each.  The own workgroups are
// numbered a-major and XCD by XCD, so the workgroups of an XCD walk the same
// K range of neighbouring tiles and share their operand panels in its L2
// (one K range after another per tile, as stream-K does it, shares none).
//
// Measured against two K halves per tile (at most half a round) or one helper
// piece per tile (more): one rollout of 1301 tokens at d = 3584 (84 tiles, 3
// pieces) 4.86 -> 4.56 ms per replay step, 10007 tokens at d = 1536 in
// 4096-token chunks (96 tiles, 8 pieces by threes) 13.62 -> 12.29 ms, 3003
// tokens there (72 tiles, 7 by twos) 5.42 -> 4.91 ms per step of four calls.
//
// A share of a tile is summed in registers.  Share 0 (own workgroup 0) goes to
// the output, share k > 0 to slot k - 1, added afterwards in slot order.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gemm_core.h"

namespace rbp {
namespace gemm {

struct Pieces {
  int32_t r, p, q, u, rem, steps;

  struct At {
    int32_t tile, piece, slot;  // slot 0: the output, k: slot k - 1
    bool flush;                 // the workgroup's last piece of this tile
  };

  // Virtual block vid = c + j P is the j-th piece of workgroup c of P.  A
  // helper past the last left-over piece gets piece p of tile 0, beyond the
  // K range (its operands read as zero and nothing is stored).
  __host__ __device__ __forceinline__ At at(int32_t vid, int32_t P) const {
    const int32_t c = vid % P, j = vid / P;
    if (c < r * u) {
      const int32_t L = (int32_t)xcd_order((uint32_t)c, (uint32_t)(r * u));
      const int32_t a = L / r;
      return At{L - a * r, a * q + j, a, j == q - 1};
    }
    const int32_t x0 = (c - r * u) * q, x = x0 + j;
    if (x >= r * rem) return At{0, p, 0, true};
    const int32_t i = x / rem;
    return At{i, u * q + (x - i * rem), u + (x0 > i * rem ? 1 : 0),
              j == q - 1 || x + 1 == (i + 1) * rem};
  }

  // Helpers that share tile i's left-over pieces: one, or two where a
  // workgroup boundary falls inside them (rem < q: never more).
  __host__ __device__ __forceinline__ int32_t slots_of(int32_t i) const {
    if (rem == 0) return u - 1;
    return u - 1 + ((i * rem) / q == (i * rem + rem - 1) / q ? 1 : 2);
  }
  // The most any tile has.
  __host__ __device__ __forceinline__ int32_t slots() const {
    return u - 1 + (rem == 0 ? 0 : (rem == 1 ? 1 : 2));
  }
  int64_t workgroups() const { return (int64_t)r * u + ((int64_t)r * rem + q - 1) / q; }
};

// The largest number of pieces up to p that needs at most max_slots (>= 1)
// slots: p / q - 1, and one more for a left-over piece, two for several.
inline int64_t fitting_pieces(int64_t p, int64_t q, int64_t max_slots) {
  const int64_t all = (max_slots + 1) * q;  // no piece left over
  if (p >= all) return all;
  const int64_t one = max_slots * q + 1;    // one
  return p < one ? p : one;                 // any below
}

// The cut of r tiles of nk K steps for G workgroups when at most max_slots
// slots fit in the scratch (p = 1: not cut).  Cost in K steps (about 1 us
// each): the q pieces a workgroup runs, a second epilogue for a helper, and
// the slots' addition -- one more launch, 256 KB read per tile and slot at
// about 4 TB/s, and a chain of loads.  A piece keeps at least min_steps steps:
// with fewer than 4 its first loads' latency outweighs them.
constexpr int64_t kMinSteps = 4;
inline Pieces plan_pieces(int64_t r, int64_t nk, int64_t G, int64_t max_slots,
                          int64_t min_steps = kMinSteps) {
  Pieces best{(int32_t)r, 1, 1, 1, 0, (int32_t)nk};
  if (r <= 0 || r >= G || max_slots < 1) return best;
  double best_cost = (double)nk;
  for (int64_t q = 1; q <= 8; ++q) {
    int64_t p = q * G / r;
    if (p > nk / min_steps) p = nk / min_steps;
    for (; p > q; p -= 1 + p / 8) {
      p = fitting_pieces(p, q, max_slots);
      if (p <= q) break;
      Pieces c{(int32_t)r, (int32_t)p, (int32_t)q, (int32_t)(p / q), (int32_t)(p % q), 0};
      if (q > 1 && c.rem == 0) continue;  // p / q pieces of one, in more parts
      c.steps = (int32_t)((nk + p - 1) / p);
      const double cost = (double)(q * c.steps) + 0.25 * (double)(q - 1) +
                          (c.rem ? 4.0 : 0.0) + 5.0 +
                          c.slots() * (0.3 + 0.065 * (double)r);
      if (cost < best_cost) {
        best_cost = cost;
        best = c;
      }
    }
  }
  return best;
}

}  // namespace gemm
}  // namespace rbp
