// Which form of a kernel a batch takes, where that follows from what the host knows of it: whole-number arithmetic on the sizes of a call,
// compiled for the host only, so that a test can ask it for any batch.
#pragma once
#include <stdint.h>

namespace hydra {
namespace rules {

constexpr int kTileTokens = 32;  // query tokens per wave tile
constexpr int kTileKeys = 64;    // keys per LDS tile

// The most items of `tiles` wave tiles that a packed batch can have: what it has for one sequence and where all have max_seqlen tokens;
// otherwise each sequence pads up to 31 tokens and less than an item.  (By an average of half of that instead, 10 sequences of 65 tokens
// with 16 heads passed for 242 items of two wave tiles and have 320.)
inline int64_t items_most(int tiles, int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t group, int32_t n_kv_heads) {
  if (batch == 1 || (int64_t)max_seqlen * batch == total_tokens) {
    const int64_t tok_tiles = ((int64_t)(total_tokens / batch) + kTileTokens - 1) / kTileTokens;
    return n_kv_heads * (int64_t)batch * ((tok_tiles * group + tiles - 1) / tiles);
  }
  const int64_t wave_tiles = ((int64_t)total_tokens + (kTileTokens - 1) * (int64_t)batch) / kTileTokens * group;
  return n_kv_heads * ((wave_tiles + (group % tiles == 0 ? 0 : tiles - 1) * (int64_t)batch) / tiles);
}

// How a packed batch is taken whose items have a compute unit each, or nearly: then the length of an item's chain of key tiles is all that
// counts (attn_fwd_direct_kernel).  A second item on a unit waits for the first, so what counts is what there can be.
// Whether its items are two wave tiles, whose keys two teams of waves divide.  This is part of the result (each team's P is
// rounded relative to a reference of its own), so it follows from the sizes that every call on the batch has in common, and calls that
// share the chip take it as well.
// us with items of four wave tiles, with loading waves as well (below), and so: one image of 577 tokens with 16 heads of 64 (160 items of
// two wave tiles) 9.45, 8.58 and 6.58; one of 1000 with 16 heads of 80 (256) 16.8, 15.4 and 12.9; requests with 28 / 4 heads of 128, of
// 558 tokens (252) 12.4, 11.3 and 8.9, of 200 (100) 7.84, 7.38 and 6.88; with 32 / 32 heads, 500 tokens (256) 11.7, 11.0 and 8.6, 544
// (288) 12.1, 11.3 and 12.3, 700 (352) 14.5, 13.2 and 16.1; several sequences, 16 heads of 64, 4 of 65 .. 300 (208) 6.90, 6.56 and 5.96,
// 10 of 65 (320) 5.2, 5.2 and 8.6, 2 of 200 .. 600 (272) 10.1, 9.3 and 11.6.  Neither pays for sequences of one key tile: 12 requests of 20
// tokens with 28 / 4 heads 5.4 and 5.9, 16 of 64 6.7 and (loading waves) 6.9.  With two key tiles a team has one, and what halving saves is
// little; at head_dim 128 the workgroups' loads of Q and their merge take it back where they fill the chip: four wave tiles and halves,
// 8 / 1 heads, of 66 tokens 96 items 6.15 and 5.93, 168 6.70 and 6.55, 204 6.99 and 7.37, 252 7.08 and 8.38, of 128 192 7.27 and 6.90, 256 7.27 and 8.14;
// 28 / 4 heads, 5 of 66 (220) 6.77 and 7.04; 64 / 8 heads, 2 of 128 (256) 6.84 and 7.01; of 192, 240 8.23 and 8.01.
inline bool more_than_a_key_tile(int32_t batch, int32_t total_tokens) { return total_tokens > (int64_t)kTileKeys * batch; }
inline bool halved_items(int32_t head_dim, int32_t batch, int32_t total_tokens, int32_t n_q_heads, int32_t n_kv_heads, unsigned compute_units) {
  const bool two_key_tiles = total_tokens <= 2 * kTileKeys * (int64_t)batch;
  return more_than_a_key_tile(batch, total_tokens) &&
         items_most(2, batch, total_tokens, 0, n_q_heads / n_kv_heads, n_kv_heads) * 4 <= (head_dim == 128 && two_key_tiles ? 3 : 4) * (int64_t)compute_units;
}
// Whether workgroups of four wave tiles get four waves more that load their tiles, so that a compute unit holds one: two images of 577
// tokens with 16 heads of 64 (160 items) 9.67 -> 8.85 us, a request of 1000 with 28 / 4 heads (224) 18.4 -> 16.2, with 32 / 32 heads
// (256) 20.0 -> 18.4; but four images (320) 13.8 -> 17.6, three requests of 500 with 28 / 4 heads (336) 14.0 -> 16.1, five of 129 with
// 32 / 32 heads (320) 8.7 -> 12.9.  One causal sequence has few long items and many short ones, which find a unit when the first are
// through: 28 / 4 heads, 1500 tokens (332) 28.3 -> 23.9; 32 / 32 heads, 1100 (288) 22.8 -> 19.3, 1300 (352) 31.0 -> 27.8, 1600 (416) 33.5 -> 35.7.
inline bool loading_waves(bool causal, int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, unsigned compute_units) {
  const int64_t most = items_most(4, batch, total_tokens, max_seqlen, n_q_heads / n_kv_heads, n_kv_heads);
  return more_than_a_key_tile(batch, total_tokens) && most * 2 <= (causal && batch == 1 ? 3 : 2) * (int64_t)compute_units;
}

}  // namespace rules
}  // namespace hydra
