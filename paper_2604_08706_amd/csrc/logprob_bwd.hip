// Backward of the policy log-probabilities (policy_logprob_bwd) and the two
// gradient products shared with the single-pass entry.
//
// Paper: App. D.2, chain rule of logp_t = z_{t,y_t} - lse_t with z_t = W h_t:
//   dz_t = dlogp_t (e_{y_t} - softmax(z_t)),  dh_t = W^T dz_t,  dW = sum_t dz_t h_t^T.
//
// Per chunk of Tc tokens:
//   1. the forward's logit product is recomputed; its epilogue writes
//      dz = -dlogp p as bf16 into dz^T [Vp][Tc] (Vp = V rounded up to 256,
//      padding zero), and a small pass overwrites each token's target entry
//      with dlogp (1 - p_{t,y_t}) from a direct dot product for z_{t,y_t};
//   2. dH[t][m] = sum_v W[v][m] dz^T[v][t]: W and dz^T read MN-major;
//   3. dW[v][m] (+)= sum_t H[t][m] dz^T[v][t]: H read MN-major, dz^T K-major.
// Every product runs on the persistent direct-load stream of gemm_dma.h (one
// 256 x 256 workgroup per CU), reading W and H in place.  The last round of
// dH's and dW's tiles is cut along K where it would leave compute units idle
// (pieces.h), and where neither product fills the chip both share one launch.
// No floating-point atomics are used, so results are bitwise reproducible.

#include "logits_epilogue.h"
#include "pieces.h"
#include "rbp_internal.h"

namespace {

using namespace rbp::lp;
using rbp::gemm::kLdsBytes;
using rbp::gemm::Tile;
using rbp::gemm::tile_stream;
using rbp::gemm::map_tile;
using rbp::gemm::xcd_block;
using rbp::gemm::Pieces;
using rbp::gemm::plan_pieces;
using rbp::gemm::Operand;
using rbp::gemm::kKMajor;
using rbp::gemm::kMNMajor;
using rbp::gemm::kKPaired;
using rbp::gemm::kOutN;

// Rows of a dW tile read, then stored back, at a time (4 values per lane each).
constexpr int kDwRows = 8;
// Longest dW row whose 256-row tile a 32-bit buffer offset spans.
constexpr int32_t kMaxBufferD = 2000000;

// Backward step 1: recompute the tile and write dz = dlogp (onehot - p) as
// bf16, vocabulary-major (Gt[v][t], the layout both later products read).
// The tile pass writes -dlogp_t p_{t,v} everywhere; the one target entry of
// each token is then overwritten by target_dz_kernel.  Masked and padding
// tokens get dz = 0 (p is evaluated against lse = +inf).

RBP_LOGITS_KERNEL void grad_logits_kernel(const uint16_t* __restrict__ W,
                                          const uint16_t* __restrict__ Hc, int64_t Tn,
                                          int32_t d, int32_t V, const int32_t* __restrict__ seq,
                                          const float* __restrict__ lse,
                                          const float* __restrict__ dlogp,
                                          uint16_t* __restrict__ Gt, int64_t ldGt,
                                          int64_t tiles_m, int64_t tiles_n) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  const Operand A{W, d, V, d};
  const Operand B{Hc, d, Tn, d};
  auto tile_of = [&](int32_t vid) {
    int32_t tm, tn;
    map_tile(vid, (int32_t)tiles_m, (int32_t)tiles_n, kGroupLogits, tm, tn);
    return Tile{tm * 256, tn * 256, 0, d};
  };
  // lse * log2 e and dlogp of this lane's token columns, loaded one tile
  // ahead (issued after an epilogue, consumed at the next one)
  float ls[GL::NI], dl[GL::NI];
  auto load_token_terms = [&](int32_t vid) {
    const Tile tile = tile_of(vid);
#pragma unroll
    for (int ni = 0; ni < GL::NI; ++ni) {
      const int64_t t = tile.n0 + GL::col_paired(ni);
      const bool valid = t < Tn && (seq == nullptr || seq[t] >= 0);
      ls[ni] = valid ? lse[t] * kLog2e : INFINITY;
      dl[ni] = valid ? dlogp[t] : 0.0f;
    }
  };
  load_token_terms((int32_t)blockIdx.x);
  const int32_t n_vid = (int32_t)(tiles_m * tiles_n);
  auto epi = [&](int32_t vid, f32x16 (&acc)[GL::MI][GL::NI]) {
    const Tile tile = tile_of(vid);
    const int32_t vlim = V - tile.m0;
    const int32_t lim = vlim - GL::row(0, 0);  // as row_off(mi, r) < lim
    // the tile's 256 x 256 corner of Gt
    const auto rGt = __builtin_amdgcn_make_buffer_rsrc(Gt + (int64_t)tile.m0 * ldGt + tile.n0, 0,
                                                       (int)(256 * ldGt * 2), 0x00020000);
    // lane l: row GL::row(0, 0), tokens 2 (l % 32) and 2 (l % 32) + 1
    const uint32_t off = (uint32_t)(GL::row(0, 0) * ldGt + GL::col_paired(0)) * 2u;
#pragma unroll
    for (int mi = 0; mi < GL::MI; ++mi) {
      if (vlim >= 256)
        dz_rows<true>(acc, ls, dl, mi, lim, rGt, off, ldGt);
      else
        dz_rows<false>(acc, ls, dl, mi, lim, rGt, off, ldGt);
    }
    if (vid + (int32_t)gridDim.x < n_vid) load_token_terms(vid + (int32_t)gridDim.x);
  };
  tile_stream<GL, kKMajor, kKPaired, kDeepLogits>(A, B, n_vid, smem, tile_of, epi);
}

// Backward step 1b, after the tile pass: the target entry of each valid
// token, dz_{t,y_t} = dlogp_t (1 - exp(z_{t,y_t} - lse_t)), with the target
// logit as one fp32 dot product h_t . W_{y_t}.  One wave per token.
__global__ void __launch_bounds__(256) target_dz_kernel(
    const uint16_t* __restrict__ Hc, const uint16_t* __restrict__ W,
    const int32_t* __restrict__ tokens, const int32_t* __restrict__ seq,
    const float* __restrict__ lse, const float* __restrict__ dlogp, int64_t Tn, int32_t d,
    int32_t V, uint16_t* __restrict__ Gt, int64_t ldGt) {
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= Tn || (seq != nullptr && seq[t] < 0)) return;
  const int32_t y = tokens[t];
  if (y < 0 || y >= V) return;
  const float z = dot_bf16_wave(Hc + t * d, W + (int64_t)y * d, d, lane);
  if (lane == 0) {
    const float p = exp2_hw((z - lse[t]) * kLog2e);
    const __bf16 g = (__bf16)(dlogp[t] * (1.0f - p));
    Gt[(int64_t)y * ldGt + t] = __builtin_bit_cast(uint16_t, g);
  }
}

// Backward step 2: dH[t][m] = c_t sum_v W[v][m] dz[t][v], with A = W and
// B = dz^T both read MN-major (m / t contiguous, k = vocabulary); c_t = 1,
// or cs[t] for the single pass.
//
// Stores one finished tile, rows scaled by c_t, into `out` laid out like dH.
__device__ __forceinline__ void store_dh(const Tile& tile, const f32x16 (&acc)[GL::MI][GL::NI],
                                         int64_t Tn, int32_t d, const float* __restrict__ cs,
                                         float* __restrict__ out) {
#pragma unroll
  for (int ni = 0; ni < GL::NI; ++ni) {
    const int64_t t = tile.n0 + GL::col(ni);
    if (t >= Tn) continue;
    const float c = cs != nullptr ? cs[t] : 1.0f;  // per-token scale of the single pass
#pragma unroll
    for (int mi = 0; mi < GL::MI; ++mi)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const int64_t m = tile.m0 + GL::row(mi, rg * 4);
        if (m < d)
          *reinterpret_cast<float4*>(out + t * d + m) =
              make_float4(c * acc[mi][ni][rg * 4 + 0], c * acc[mi][ni][rg * 4 + 1],
                          c * acc[mi][ni][rg * 4 + 2], c * acc[mi][ni][rg * 4 + 3]);
      }
  }
}

// Whole rounds: blocks 0 .. n_vid - 1 of the launch over every tile, the whole
// vocabulary per tile.
RBP_LOGITS_KERNEL void dhidden_kernel(const uint16_t* __restrict__ W,
                                      const uint16_t* __restrict__ Gt, int64_t ldGt, int64_t Tn,
                                      int32_t d, int32_t V, const float* __restrict__ cs,
                                      float* __restrict__ dH, int64_t tiles_m, int64_t tiles_n,
                                      int32_t n_vid) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  const int64_t T256 = (Tn + 255) / 256 * 256;
  const Operand A{W, d, d, V};          // (m = hidden unit, k = vocab): W[v][m]
  const Operand B{Gt, ldGt, T256, V};   // (n = token, k = vocab): Gt[v][t]
  auto tile_of = [&](int32_t vid) {
    int32_t tm, tn;
    map_tile(vid, (int32_t)tiles_m, (int32_t)tiles_n, kGroupGrad, tm, tn);
    return Tile{tm * 256, tn * 256, 0, V};
  };
  auto epi = [&](int32_t vid, f32x16 (&acc)[GL::MI][GL::NI]) {
    store_dh(tile_of(vid), acc, Tn, d, cs, dH);
  };
  tile_stream<GL, kMNMajor, kMNMajor, kDeepDh>(A, B, n_vid, smem, tile_of, epi);
}

// Tile i of the r tiles of a last round, blocks base .. base + r - 1 of the
// launch over every tile: XCD by XCD, so that neighbouring i are neighbours.
__device__ __forceinline__ void last_round_tile(int32_t i, int32_t r, int32_t base,
                                                int64_t tiles_m, int64_t tiles_n, int32_t& tm,
                                                int32_t& tn) {
  map_tile(base + (int32_t)xcd_block((uint32_t)i, (uint32_t)r), (int32_t)tiles_m,
           (int32_t)tiles_n, kGroupGrad, tm, tn);
}

// The last round of a dhidden launch: its r tiles (blocks base .. base + r - 1
// of the launch over every tile), fewer than there are compute units, cut along
// the vocabulary so that every unit has work (pieces.h).  A workgroup's accumulators
// are carried from piece to piece of a tile; a tile's first share goes to dH
// and the others to their slots of `part`, arrays laid out like dH that
// part_add_dh_kernel adds in order.
struct DhArgs {
  const uint16_t* W;
  const uint16_t* Gt;
  int64_t ldGt, Tn;
  int32_t d, V;
  const float* cs;
  float* dH;
  int64_t tiles_m, tiles_n;
  int32_t base;
  Pieces pc;
  float* part;
  int64_t slot_floats;
};

__device__ __forceinline__ void dhidden_pieces(const DhArgs& g, uint8_t* smem, int32_t wg,
                                               int32_t n_wg) {
  const int64_t T256 = (g.Tn + 255) / 256 * 256;
  const Operand A{g.W, g.d, g.d, g.V};        // (m = hidden unit, k = vocab): W[v][m]
  const Operand B{g.Gt, g.ldGt, T256, g.V};   // (n = token, k = vocab): Gt[v][t]
  auto tile_of = [&](int32_t vid) {
    const Pieces::At a = g.pc.at(vid, n_wg);
    int32_t tm, tn;
    last_round_tile(a.tile, g.pc.r, g.base, g.tiles_m, g.tiles_n, tm, tn);
    // every piece spans `steps` steps; rows past V read as zero
    const int32_t kb = a.piece * g.pc.steps * 64;
    return Tile{tm * 256, tn * 256, kb, kb + g.pc.steps * 64};
  };
  auto epi = [&](int32_t vid, f32x16 (&acc)[GL::MI][GL::NI]) -> bool {
    const Pieces::At a = g.pc.at(vid, n_wg);
    if (!a.flush) return false;  // the tile's next piece follows on this workgroup
    if (a.piece < g.pc.p)
      store_dh(tile_of(vid), acc, g.Tn, g.d, g.cs,
               a.slot == 0 ? g.dH : g.part + (a.slot - 1) * g.slot_floats);
    return true;
  };
  tile_stream<GL, kMNMajor, kMNMajor, kDeepDh>(A, B, g.pc.q * n_wg, smem, tile_of, epi, wg, n_wg);
}

RBP_LOGITS_KERNEL void dhidden_pieces_kernel(DhArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  dhidden_pieces(g, smem, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

// dH += its tiles' slots of `part`, in slot order; one block per (tile, 4
// tokens), 16 bytes per lane.
__global__ void __launch_bounds__(256) part_add_dh_kernel(float* __restrict__ dH,
                                                          const float* __restrict__ part,
                                                          int64_t slot_floats, int32_t base,
                                                          Pieces pc, int64_t tiles_m,
                                                          int64_t tiles_n, int32_t d,
                                                          int64_t Tn) {
  const int32_t i = (int32_t)blockIdx.x;
  int32_t tm, tn;
  last_round_tile(i, pc.r, base, tiles_m, tiles_n, tm, tn);
  const int64_t t = (int64_t)tn * 256 + blockIdx.y * 4 + (threadIdx.x >> 6);
  const int32_t m = tm * 256 + (threadIdx.x & 63) * 4;
  if (t >= Tn || m >= d) return;  // d % 8 == 0: a float4 never straddles the edge
  float4* dst = reinterpret_cast<float4*>(dH + t * d + m);
  float4 o = *dst;
  const int32_t n = pc.slots_of(i);
#pragma unroll 4
  for (int32_t k = 0; k < n; ++k) {
    const float4 p = *reinterpret_cast<const float4*>(part + k * slot_floats + t * d + m);
    o.x += p.x;
    o.y += p.y;
    o.z += p.z;
    o.w += p.w;
  }
  *dst = o;
}

// Stores one finished dW tile, adding the previous values when `accumulate`.
//
// A lane holds one column m (kOutN), so 32 lanes cover one 128-byte line of a
// row and an instruction two whole lines.  With runs of four m per lane
// (16-byte accesses, 32 rows of 32 bytes each) the address unit took every
// line four times, and a tile's read-modify-write of 512 KB cost about 30 us
// beside its K loop (1.5 us a step): dW at d = 3584, V = 152064 took 2.05 ms
// for 1301 tokens, 1.66 ms this way, and 14.50 / 14.45 ms for 16384; without
// accumulation into d = 1536, V = 151936, 4096 tokens 1.12 -> 0.96 ms.
//
// Rows go through a buffer resource over the tile, one offset per lane and
// 32-column block; columns past d point beyond the range (loads read 0, stores
// are dropped).  Inside the matrix the row is the scalar offset.  In a tile
// that ends past the vocabulary or past d (kTail) it is part of the lane's
// offset, which the range check covers, so that rows past V are dropped too,
// and blocks of columns past d are left out (d = 64: 6 of 8).
template <bool kTail>
__device__ __forceinline__ void dw_rows(const f32x16 (&acc)[GL::MI][GL::NI],
                                        float* __restrict__ dW, const Tile& tile, int32_t d,
                                        int32_t V, int accumulate) {
  const int64_t left = V - tile.n0, rows = left < 256 ? left : 256;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
      uniform_ptr(dW + (int64_t)tile.n0 * d + tile.m0), 0,
      (int)(((rows - 1) * d + (d - tile.m0)) * 4), 0x00020000);
  auto lane_offset = [&](int mi) {
    const int m = GL::out_m(mi) + GL::lane_m();
    return tile.m0 + m < d ? (uint32_t)(GL::lane_n() * d + m) * 4u : rbp::gemm::kOutOfRange;
  };
  if constexpr (kTail) {
#pragma unroll
    for (int mi = 0; mi < GL::MI; ++mi) {
      if (tile.m0 + GL::out_m(mi) >= d) continue;
      const uint32_t at = lane_offset(mi);
#pragma unroll
      for (int ni = 0; ni < GL::NI; ++ni) {
        float o[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
          o[r] = !accumulate ? 0.0f
                             : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                   rsrc, at + GL::out_n(ni, r) * d * 4, 0, 0));
#pragma unroll
        for (int r = 0; r < 16; ++r)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[mi][ni][r] + o[r]), rsrc,
                                                at + GL::out_n(ni, r) * d * 4, 0, 0);
        asm volatile("" ::: "memory");
      }
    }
    return;
  }
  uint32_t at[GL::MI];
#pragma unroll
  for (int mi = 0; mi < GL::MI; ++mi) at[mi] = lane_offset(mi);
#pragma unroll
  for (int ni = 0; ni < GL::NI; ++ni)
#pragma unroll
    for (int rb = 0; rb < 16; rb += kDwRows) {
      // the previous values of kDwRows rows are loaded before any of them is
      // stored back, so the tile waits for memory four times (8 rows; 4 rows
      // time the same)
      float o[kDwRows][GL::MI];
#pragma unroll
      for (int k = 0; k < kDwRows; ++k)
#pragma unroll
        for (int mi = 0; mi < GL::MI; ++mi)
          o[k][mi] = !accumulate ? 0.0f
                                 : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                       rsrc, at[mi], GL::out_n(ni, rb + k) * d * 4, 0));
#pragma unroll
      for (int k = 0; k < kDwRows; ++k)
#pragma unroll
        for (int mi = 0; mi < GL::MI; ++mi)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[mi][ni][rb + k] + o[k][mi]),
                                                rsrc, at[mi], GL::out_n(ni, rb + k) * d * 4, 0);
      // keeps the next rows' loads below these stores (the compiler would
      // otherwise hoist them all)
      asm volatile("" ::: "memory");
    }
}

// Backward step 3: dW[v][m] (+)= sum_t H[t][m] dz[t][v], with A = H read
// MN-major (m contiguous, k = token) and B = dz^T K-major (rows v, k = token).
// The launch covers the first n_vid of the tiles of the vocabulary range
// [tn_off, tn_off + tiles_n), or (kPieces) the last round of them, blocks base
// .. base + r - 1 of the launch over every tile, cut along the tokens (Pieces)
// where it would leave compute units idle: a tile's first share updates dW, the
// others write their raw sums to slots of `part` (slot k of tile i: a 256 x 256
// fp32 block, [v][m]), which part_add_kernel adds afterwards.  Columns of dz^T
// past Tn are finite (the single pass) or zero, and meet zero rows of H.
struct DwArgs {
  const uint16_t* Hc;
  const uint16_t* Gt;
  int64_t ldGt, Tn;
  int32_t d, V;
  float* dW;
  int32_t accumulate;
  int64_t tiles_m, tiles_n, tn_off;
  int32_t n_vid;       // whole tiles
  int32_t base;        // kPieces
  Pieces pc;
  float* part;
};

// Tile i of the r tiles of a last round, as dhidden's last_round_tile.
__device__ __forceinline__ void last_dw_tile(int32_t i, const DwArgs& g, int32_t& tm,
                                             int32_t& tn) {
  map_tile(g.base + (int32_t)xcd_block((uint32_t)i, (uint32_t)g.pc.r), (int32_t)g.tiles_m,
           (int32_t)g.tiles_n, kGroupDw, tm, tn);
}

template <bool kPieces>
__device__ __forceinline__ void dweight_tiles(const DwArgs& g, uint8_t* smem, int32_t wg,
                                              int32_t n_wg) {
  const int64_t Tn = g.Tn, tn_off = g.tn_off;
  const int32_t d = g.d, V = g.V, accumulate = g.accumulate;
  float* dW = g.dW;
  const int64_t T8 = (Tn + 7) / 8 * 8;
  const Operand A{g.Hc, d, d, Tn};        // (m = hidden unit, k = token): H[t][m]
  const Operand B{g.Gt, g.ldGt, V, T8};   // (n = vocab, k = token): Gt[v][t]
  auto tile_of = [&](int32_t vid) {
    int32_t tm, tn, kb = 0, ke = (int32_t)Tn;
    if constexpr (kPieces) {
      const Pieces::At a = g.pc.at(vid, n_wg);
      last_dw_tile(a.tile, g, tm, tn);
      kb = a.piece * g.pc.steps * 64;  // tokens past Tn read as zero
      ke = kb + g.pc.steps * 64;
    } else {
      map_tile(vid, (int32_t)g.tiles_m, (int32_t)g.tiles_n, kGroupDw, tm, tn);
    }
    return Tile{tm * 256, (tn + (int32_t)tn_off) * 256, kb, ke};
  };
  auto store = [&](int32_t vid, f32x16 (&acc)[GL::MI][GL::NI]) {
    const Tile tile = tile_of(vid);
    if (d <= kMaxBufferD) {
      if (tile.n0 + 256 <= V && tile.m0 + 256 <= d)
        dw_rows<false>(acc, dW, tile, d, V, accumulate);
      else
        dw_rows<true>(acc, dW, tile, d, V, accumulate);
      return;
    }
#pragma unroll
    for (int ni = 0; ni < GL::NI; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t v = tile.n0 + GL::out_n(ni, r) + GL::lane_n();
        if (v >= V) continue;
#pragma unroll
        for (int mi = 0; mi < GL::MI; ++mi) {
          const int64_t m = tile.m0 + GL::out_m(mi) + GL::lane_m();
          if (m >= d) continue;
          float* dst = dW + v * d + m;
          *dst = accumulate ? acc[mi][ni][r] + *dst : acc[mi][ni][r];
        }
      }
  };
  if constexpr (kPieces) {
    auto epi = [&](int32_t vid, f32x16 (&acc)[GL::MI][GL::NI]) -> bool {
      const Pieces::At a = g.pc.at(vid, n_wg);
      if (!a.flush) return false;  // the tile's next piece follows on this workgroup
      if (a.piece >= g.pc.p) return true;
      if (a.slot == 0) {
        store(vid, acc);
        return true;
      }
      float* blk = g.part + ((int64_t)(a.slot - 1) * g.pc.r + a.tile) * 65536;
#pragma unroll
      for (int ni = 0; ni < GL::NI; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int mi = 0; mi < GL::MI; ++mi)
            blk[(GL::out_n(ni, r) + GL::lane_n()) * 256 + GL::out_m(mi) + GL::lane_m()] =
                acc[mi][ni][r];
      return true;
    };
    tile_stream<GL, kMNMajor, kKMajor, kDeepDw, kOutN>(A, B, g.pc.q * n_wg, smem, tile_of, epi, wg,
                                                       n_wg);
  } else {
    tile_stream<GL, kMNMajor, kKMajor, kDeepDw, kOutN>(A, B, g.n_vid, smem, tile_of, store, wg,
                                                       n_wg);
  }
}

template <bool kPieces>
RBP_LOGITS_KERNEL void dweight_kernel(DwArgs g) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  dweight_tiles<kPieces>(g, smem, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

// Both products of a small batch in one launch: workgroups below n_dw take a
// dW tile each, the others dhidden's pieces.  Neither needs the other's result
// and neither fills the chip, so together they take as long as the longer one
// (each is bound by the latency of its own chain of K steps and its stores).
RBP_LOGITS_KERNEL void grad_both_kernel(DwArgs w, DhArgs h, int32_t n_dw) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[kLdsBytes];
  const int32_t b = (int32_t)blockIdx.x;
  if (b < n_dw)
    dweight_tiles<false>(w, smem, b, n_dw);
  else
    dhidden_pieces(h, smem, b - n_dw, (int32_t)gridDim.x - n_dw);
}

// dW += the slots of the tiles of a last round, in slot order; one block per
// (tile, 4 vocabulary rows), 16 bytes per lane.
__global__ void __launch_bounds__(256) part_add_kernel(DwArgs g) {
  const int32_t i = (int32_t)blockIdx.x;
  int32_t tm, tn;
  last_dw_tile(i, g, tm, tn);
  const int32_t vl = (int32_t)blockIdx.y * 4 + (threadIdx.x >> 6), ml = (threadIdx.x & 63) * 4;
  const int64_t v = ((int64_t)tn + g.tn_off) * 256 + vl;
  const int32_t m = tm * 256 + ml;
  if (v >= g.V || m >= g.d) return;  // d % 8 == 0: a float4 never straddles the edge
  float4* dst = reinterpret_cast<float4*>(g.dW + v * g.d + m);
  float4 o = *dst;
  const int32_t n = g.pc.slots_of(i);
#pragma unroll 4
  for (int32_t k = 0; k < n; ++k) {
    const float4 p = *reinterpret_cast<const float4*>(
        g.part + ((int64_t)k * g.pc.r + i) * 65536 + vl * 256 + ml);
    o.x += p.x;
    o.y += p.y;
    o.z += p.z;
    o.w += p.w;
  }
  *dst = o;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(float* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    p[i] = 0.0f;
}



inline void launch_part_add(const DhArgs& g, hipStream_t s) {
  hipLaunchKernelGGL(part_add_dh_kernel, dim3((unsigned)g.pc.r, 64), dim3(256), 0, s, g.dH, g.part,
                     g.slot_floats, g.base, g.pc, g.tiles_m, g.tiles_n, g.d, g.Tn);
}

// Backward workspace carving: dz^T [Vp][T256] bf16, then scratch for partial
// sums, [T256][d] fp32 at least.
struct BwdWs {
  uint16_t* Gt;
  float* scratch;
  size_t scratch_at;  // byte offset of scratch
  size_t bytes;
};
BwdWs carve_bwd(void* base, int64_t Tc, int32_t d, int32_t V) {
  rbp::WsCarver c(base);
  const int64_t T256 = round256(Tc < 1 ? 1 : Tc), Vp = round256(V);
  BwdWs w;
  w.Gt = c.take<uint16_t>((size_t)Vp * (size_t)T256);
  w.scratch = c.take<float>((size_t)T256 * (size_t)d);
  w.scratch_at = c.used - sizeof(float) * (size_t)T256 * (size_t)d;
  w.bytes = rbp::align_up(c.used, 256);
  return w;
}
}  // namespace

size_t rbp::logprob_bwd_ws(int64_t Tc, int32_t d, int32_t V) {
  const int64_t T256 = round256(Tc < 1 ? 1 : Tc);
  const int32_t dd = d < 1 ? 1 : d;
  const BwdWs w = carve_bwd(nullptr, T256, dd, V);
  // Planned with pieces of 8 steps, where a launch cuts down to 4 (and the single
  // pass asks for 4), for the sake of the size alone: heads of up to 1024 words
  // then ask for exactly dz^T and one dhidden, which callers may have counted
  // on.  It costs them time, not results: 256 tokens of d = 64, V = 1000 take
  // 29.8 us so and 25.7 with 575 KB more, which a caller may give; d = 128,
  // V = 2048 33.1 with the 256 KB asked for, 30.0 with 1.1 MB, 41.9 with none.
  // From d = 512 on both plans ask for the most a chunk may.
  return w.bytes + dhidden_extra(T256, dd, V, w.bytes - w.scratch_at, w.bytes,
                                 carve_bwd(nullptr, T256 + 256, dd, V).bytes, 8);
}

namespace {

// The cut of dW's last round, tiles % G of its tiles, along the tokens.  Only
// where it fills at most three quarters of the chip: past that the pieces'
// extra epilogues, each a read-modify-write of 512 KB, eat what the idle units
// would give (and the busy ones run at a higher clock without them).
Pieces plan_dweight(int64_t tiles, int64_t nk, int64_t G, const float* scratch,
                    int64_t scratch_floats) {
  const int64_t r = tiles % G;
  const int64_t slots = scratch == nullptr || r == 0 || 4 * r > 3 * G
                            ? 0
                            : scratch_floats / (r * 65536);
  return plan_pieces(r, nk, G, slots, 8);
}

}  // namespace

void rbp::launch_dweight(const uint16_t* Hc, const uint16_t* Gt, int64_t ldGt, int64_t Tn,
                         int32_t d, int32_t V, float* dW, int accumulate, int64_t tn_begin,
                         int64_t tn_end, hipStream_t s, float* scratch, int64_t scratch_floats) {
  const int64_t tiles_d = rbp::ceil_div(d, 256), tiles_n = tn_end - tn_begin;
  if (tiles_n <= 0) return;
  const int64_t tiles = tiles_d * tiles_n;
  const int64_t G = rbp::gemm::stream_grid(int64_t(1) << 30, device_cus());  // one round
  const Pieces pc = plan_dweight(tiles, rbp::ceil_div(Tn, 64), G, scratch, scratch_floats);
  const int64_t n_main = pc.p > 1 ? tiles - pc.r : tiles;
  const DwArgs g{Hc,      Gt,       ldGt,            Tn, d,  V,      dW, accumulate, tiles_d,
                 tiles_n, tn_begin, (int32_t)n_main, (int32_t)n_main, pc, scratch};
  if (n_main > 0)
    hipLaunchKernelGGL(dweight_kernel<false>, dim3(rbp::gemm::stream_grid(n_main, device_cus())),
                       dim3(GL::kThreads), 0, s, g);
  if (pc.p > 1) {
    hipLaunchKernelGGL(dweight_kernel<true>, dim3((unsigned)pc.workgroups()),
                       dim3(GL::kThreads), 0, s, g);
    hipLaunchKernelGGL(part_add_kernel, dim3((unsigned)pc.r, 64), dim3(256), 0, s, g);
  }
}

void rbp::launch_dhidden(const uint16_t* W, const uint16_t* Gt, int64_t ldGt, int64_t Tn,
                         int32_t d, int32_t V, float* dhidden_c, hipStream_t s, float* scratch,
                         int64_t scratch_floats, const float* cs) {
  const int64_t tiles_d = rbp::ceil_div(d, 256), tiles_t = rbp::ceil_div(Tn, 256);
  const int64_t tiles = tiles_d * tiles_t;
  const int64_t G = rbp::gemm::stream_grid(int64_t(1) << 30, device_cus());  // one round
  const int64_t slot_floats = Tn * d;
  const int64_t r = tiles % G;
  const Pieces pc = plan_pieces(r, rbp::ceil_div(V, 64), G, scratch_floats / slot_floats);
  const int64_t n_main = pc.p > 1 ? tiles - r : tiles;
  if (n_main > 0)
    hipLaunchKernelGGL(dhidden_kernel, dim3(rbp::gemm::stream_grid(n_main, device_cus())),
                       dim3(GL::kThreads), 0, s, W, Gt, ldGt, Tn, d, V, cs, dhidden_c, tiles_d,
                       tiles_t, (int32_t)n_main);
  if (pc.p > 1) {
    const DhArgs g{W,       Gt,      ldGt,            Tn, d,       V,          cs, dhidden_c,
                   tiles_d, tiles_t, (int32_t)n_main, pc, scratch, slot_floats};
    hipLaunchKernelGGL(dhidden_pieces_kernel, dim3((unsigned)pc.workgroups()),
                       dim3(GL::kThreads), 0, s, g);
    launch_part_add(g, s);
  }
}

bool rbp::launch_both_products(const uint16_t* Hc, const uint16_t* W, const uint16_t* Gt,
                               int64_t ldGt, int64_t Tn, int32_t d, int32_t V, float* dhidden_c,
                               float* dW, int accumulate, hipStream_t s, float* scratch,
                               int64_t scratch_floats, const float* cs) {
  const int64_t tiles_d = rbp::ceil_div(d, 256), tiles_t = rbp::ceil_div(Tn, 256);
  const int64_t tiles_v = rbp::ceil_div(V, 256);
  const int64_t G = rbp::gemm::stream_grid(int64_t(1) << 30, device_cus());
  // one dW tile per workgroup, the rest of a round for dhidden; whole groups
  // of 8 keep a workgroup's number and its XCD together
  const int64_t n_dw = (tiles_d * tiles_v + 7) / 8 * 8, r = tiles_d * tiles_t;
  if (n_dw >= G || r > G - n_dw) return false;
  const int64_t slot_floats = Tn * d, max_slots = scratch_floats / slot_floats;
  const int64_t nk_v = rbp::ceil_div(V, 64), nk_t = rbp::ceil_div(Tn, 64);
  const Pieces alone = plan_pieces(r, nk_v, G, max_slots);
  const Pieces pc = plan_pieces(r, nk_v, G - n_dw, max_slots);
  // In K steps (about 1 us): the two in turn, each with a launch and an
  // epilogue of about 12, against the longer of the two.
  const Pieces dw_alone = plan_dweight(tiles_d * tiles_v, nk_t, G, scratch, scratch_floats);
  const int64_t in_turn = (int64_t)dw_alone.q * dw_alone.steps + 12 + (dw_alone.p > 1 ? 6 : 0) +
                          (int64_t)alone.q * alone.steps + 12;
  const int64_t dw = nk_t + 12, dh = (int64_t)pc.q * pc.steps + 12;
  if ((dw > dh ? dw : dh) >= in_turn) return false;
  const DwArgs w{Hc,      Gt, ldGt, Tn, d, V, dW, accumulate, tiles_d,
                 tiles_v, 0,  (int32_t)(tiles_d * tiles_v), 0, dw_alone, nullptr};
  const DhArgs h{W,       Gt,      ldGt, Tn, d,       V,          cs, dhidden_c,
                 tiles_d, tiles_t, 0,    pc, scratch, slot_floats};
  hipLaunchKernelGGL(grad_both_kernel, dim3((unsigned)(n_dw + pc.workgroups())),
                     dim3(GL::kThreads), 0, s, w, h, (int32_t)n_dw);
  if (pc.p > 1) launch_part_add(h, s);
  return true;
}

size_t rbp::dhidden_extra(int64_t T256, int32_t d, int32_t V, size_t free_bytes, size_t base,
                          size_t next, int64_t min_steps) {
  // sized for the 256 compute units of an MI355X, 64 MiB of partial sums at
  // most (one 256 x 256 block per unit)
  constexpr int64_t kUnits = 256;
  const int64_t slot = T256 * (int64_t)d * 4;
  const int64_t tiles = rbp::ceil_div(d, 256) * (T256 / 256);
  const Pieces pc = plan_pieces(tiles % kUnits, rbp::ceil_div(V, 64), kUnits,
                                (kUnits << 18) / slot, min_steps);
  const size_t want = (size_t)(pc.slots() * slot);
  if (want <= free_bytes) return 0;
  const size_t extra = align_up(want - free_bytes, 256);
  return base + extra < next ? extra : next - base - 256;
}

void rbp::launch_grad_products(const uint16_t* Hc, const uint16_t* W, const uint16_t* Gt,
                               int64_t ldGt, int64_t Tn, int32_t d, int32_t V, float* dhidden_c,
                               float* dW, int accumulate, hipStream_t s, float* scratch,
                               int64_t scratch_floats) {
  if (Tn == 0) {
    if (!accumulate) {
      const int64_t n = (int64_t)V * d;
      int64_t blocks = rbp::ceil_div(n, 256);
      if (blocks > 65536) blocks = 65536;
      hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, s, dW, n);
    }
    return;
  }
  if (launch_both_products(Hc, W, Gt, ldGt, Tn, d, V, dhidden_c, dW, accumulate, s, scratch,
                           scratch_floats))
    return;
  launch_dhidden(W, Gt, ldGt, Tn, d, V, dhidden_c, s, scratch, scratch_floats);
  // the scratch is free again once dhidden's sum has read it
  launch_dweight(Hc, Gt, ldGt, Tn, d, V, dW, accumulate, 0, round256(V) / 256, s, scratch,
                 scratch_floats);
}

extern "C" int policy_logprob_bwd(const uint16_t* hidden, const uint16_t* W,
                                  const int32_t* tokens, const int32_t* seq_of_token,
                                  const float* lse, const float* dlogp, int64_t T, int32_t d,
                                  int32_t V, float* dhidden, float* dW, int accumulate_dW,
                                  void* ws, size_t ws_bytes, void* stream) {
  rbp::clear_error();
  RBP_REQUIRE(T >= 0 && d >= 1 && V >= 1, RBP_EINVAL,
              "policy_logprob_bwd: need T >= 0, d >= 1, V >= 1");
  RBP_REQUIRE(d % 8 == 0, RBP_EUNSUPPORTED, "policy_logprob_bwd: d %% 8 != 0 (d = %d)", d);
  RBP_REQUIRE(W && dW, RBP_EINVAL, "policy_logprob_bwd: null pointer");
  RBP_REQUIRE(T == 0 || (hidden && tokens && lse && dlogp && dhidden), RBP_EINVAL,
              "policy_logprob_bwd: null pointer");
  hipStream_t s = rbp::as_stream(stream);
  if (T == 0) {
    rbp::launch_grad_products(nullptr, W, nullptr, 0, 0, d, V, nullptr, dW, accumulate_dW, s,
                              nullptr, 0);
    RBP_CHECK_LAUNCH("policy_logprob_bwd");
    return RBP_OK;
  }
  // largest chunk (multiple of 256 tokens) whose workspace fits
  int64_t Tc = 0;
  if (ws) {
    // chunks of at most 2^21 tokens keep every per-tile byte range of dz^T
    // (256 rows x Tc x 2 bytes) inside a 32-bit buffer offset
    int64_t lo = 256, hi = round256(T) < (int64_t(1) << 21) ? round256(T) : (int64_t(1) << 21);
    if (carve_bwd(nullptr, lo, d, V).bytes <= ws_bytes) {
      while (lo < hi) {  // largest multiple of 256 in [lo, hi] that fits
        const int64_t mid = (lo + hi + 256) / 512 * 256;
        if (carve_bwd(nullptr, mid, d, V).bytes <= ws_bytes) lo = mid; else hi = mid - 256;
      }
      Tc = lo;
    }
  }
  RBP_REQUIRE(Tc >= 256, RBP_EWORKSPACE,
              "policy_logprob_bwd: workspace of %zu bytes holds no 256-token chunk (needs %zu)",
              ws_bytes, carve_bwd(nullptr, 256, d, V).bytes);
  const BwdWs w = carve_bwd(ws, Tc, d, V);
  const int64_t tiles_v = round256(V) / 256;
  const int n_cu = device_cus();
  for (int64_t t0 = 0; t0 < T; t0 += Tc) {
    const int64_t Tn = (T - t0) < Tc ? (T - t0) : Tc;
    const int64_t tiles_t = rbp::ceil_div(Tn, 256);
    const uint16_t* Hc = hidden + t0 * d;
    hipLaunchKernelGGL(grad_logits_kernel, dim3(rbp::gemm::stream_grid(tiles_v * tiles_t, n_cu)),
                       dim3(GL::kThreads), 0, s, W, Hc, Tn, d, V,
                       seq_of_token ? seq_of_token + t0 : nullptr, lse + t0, dlogp + t0, w.Gt,
                       Tc, tiles_v, tiles_t);
    hipLaunchKernelGGL(target_dz_kernel, dim3(rbp::ceil_div(Tn, 4)), dim3(256), 0, s, Hc, W,
                       tokens + t0, seq_of_token ? seq_of_token + t0 : nullptr, lse + t0,
                       dlogp + t0, Tn, d, V, w.Gt, Tc);
    rbp::launch_grad_products(Hc, W, w.Gt, Tc, Tn, d, V, dhidden + t0 * d, dW,
                              (accumulate_dW || t0 > 0) ? 1 : 0, s, w.scratch,
                              (int64_t)((ws_bytes - w.scratch_at) / sizeof(float)));
  }
  RBP_CHECK_LAUNCH("policy_logprob_bwd");
  return RBP_OK;
}
