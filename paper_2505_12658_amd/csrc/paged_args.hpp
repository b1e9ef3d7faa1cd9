// Arguments of the paged attention kernels, and how long contexts are cut into shares.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_tiles.hpp"

namespace hydra {
namespace paged {

constexpr int kRows = 32;          // new tokens (or packed rows) per wave tile
constexpr int kWavesPerGroup = 4;  // wave tiles per workgroup
constexpr int kNeverOrdered = 0x7fffffff;

struct PagedArgs {
  const uint16_t* q;        // [total_q, n_q_heads, D] with token stride
  uint16_t* out;            // [total_q, n_q_heads, D] contiguous
  int64_t q_stride;         // elements per token
  const uint16_t* k_cache;  // [num_blocks, block_size, n_kv_heads, D]
  const uint16_t* v_cache;
  const int32_t* block_tables;  // [batch, max_blocks_per_seq]
  const int32_t* cu_seqlens_q;  // [batch + 1]
  const int32_t* kv_lens;       // [batch]
  int32_t max_blocks_per_seq;
  int32_t num_blocks;
  int32_t block_shift;  // log2(block_size)
  int32_t n_q_heads;
  int32_t n_kv_heads;
  int32_t group;     // n_q_heads / n_kv_heads
  float scale_log2;  // softmax_scale * log2(e)
  // Packed-rows form, long contexts split over workgroups: a context is cut into up to n_splits shares, all of
  // (nearly) the same length, and no more than 1 << least_log2 half tiles (32 keys each) ask for (share_plan); n_splits
  // workgroups per (request, KV head), one per share.  A context of one share is done by its first workgroup, which
  // writes `out` itself (the others leave at once); of a longer one every share leaves a partial result in `partials`, and the combine kernel merges them.  n_splits == 1: never split.
  int32_t n_splits;
  int32_t least_log2;
  float* partials;  // [batch, n_kv_heads, n_splits] records of kPartialFloats<D> floats
  int32_t batch;
  int32_t n_tile_wgs;  // workgroups that the grid has for the wave-tile form (an upper bound from the host)
  int32_t order_keys;  // a hybrid batch with a context of more keys is taken by its contexts (0: whatever they are, kNeverOrdered: not at all)
};

// One partial result of the packed-rows form: per row (32 rows) the maximum and the sum, then the
// unnormalised output rows [32][D] (only the first q_len * group rows are written and read).
template <int D>
constexpr int kPartialFloats = 2 * kRows + kRows * D;

// How a context of n_halves half tiles is cut: `shares` shares of `per` half tiles (the last one may be shorter); as few as
// keep a share to 1 << least_log2 half tiles, at most n_splits.
// The context decides, not the width of the block table, which is all that the host knows and may be far wider: with the
// share's size taken from a table of 32 768 keys 8 requests of 16 384 keys took 60.1 us instead of 45.0, 4 of 300 .. 1500 13.2
// instead of 7.9, 12 of 1000 .. 3731 36.7 instead of 15.2.  (A size for the whole batch, from the longest of kv_lens read by
// every workgroup, cost each of the two kernels another 0.3 us of latency.)
__device__ __forceinline__ void share_plan(int n_halves, int n_splits, int least_log2, int& per, int& shares) {
  per = n_halves;
  shares = 1;
  const int most = (n_halves + (1 << least_log2) - 1) >> least_log2;
  const int k = n_splits < most ? n_splits : most;
  if (k < 2) return;
  per = quotient(n_halves + k - 1, k);
  shares = quotient(n_halves + per - 1, per);
}
// half tiles [begin, end) of share s (empty past the last share)
__device__ __forceinline__ void split_range(int n_halves, int per, int s, int& begin, int& end) {
  begin = s * per < n_halves ? s * per : n_halves;
  end = begin + per < n_halves ? begin + per : n_halves;
}

}  // namespace paged
}  // namespace hydra
