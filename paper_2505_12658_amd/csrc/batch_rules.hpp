// Which form of a kernel a batch takes, where that follows from what the host knows of it: arithmetic on the sizes of a call,
// compiled for the host only, so that a test can ask it for any batch.
#pragma once
#include <stdint.h>

namespace hydra {
namespace rules {

constexpr int kTileTokens = 32;  // query tokens per wave tile
constexpr int kTileKeys = 64;    // keys per LDS tile
constexpr int kUnits = 256;      // compute units

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

// A hybrid batch of the paged call, as far as the host knows it: the lengths are on the device.
struct Hybrid {
  int32_t batch, total_q, max_q_len;  // requests; new tokens in all and of the longest request
  int32_t group, n_kv_heads, n_splits;
  int64_t table_keys;
};
constexpr int kChainTiles = 4;   // wave tiles of a chain
constexpr int kWideMost = 128;   // requests of a batch that wide workgroups take
constexpr int kTrailing = 32;    // places at the end of a wide grid that are chains at least, if not all places fit the grid
// Requests of this many new tokens and more are chunks, in chains; the others are decode steps, of n_splits workgroups per KV head each.
inline int32_t least_chunk(int32_t group) { return kTileTokens / group + 1; }
inline int64_t chains_of(int64_t tokens, int32_t group) { return ((tokens + kTileTokens - 1) / kTileTokens * group + kChainTiles - 1) / kChainTiles; }
// The most places, one for every chain and step_places for every decode step, that such a batch can have if every request has a new token
// and one has max_q_len.  Two bounds, each linear in the number of other chunks: all tokens that the chunks can have, each padded; and a chain or more for
// every chunk of the least length, and what the tokens beyond that can add at the least price of a chain more.
inline int64_t places_most(const Hybrid& b, double step_places) {
  const int64_t g = b.group, least = least_chunk(b.group), spare_all = (int64_t)b.total_q - b.batch - (b.max_q_len - 1), spare = spare_all > 0 ? spare_all : 0;
  const int64_t others = b.batch - 1, fit = least > 1 ? spare / (least - 1) : others, most = fit < others ? fit : others;
  const int64_t price = (least + kTileTokens - 1) / kTileTokens * kTileTokens + 1 - least;  // tokens from the least chunk to its next wave tiles
  double by_tokens = 0, by_chunks = 0;
  const int64_t ends[] = {0, most > 0 ? 1 : 0, most};
  for (int64_t k : ends) {
    const double steps = (double)(others - k) * b.n_kv_heads * step_places;
    const int64_t n = k + 1, tokens = (int64_t)b.total_q - (b.batch - n);
    const double padded = (double)(((tokens + (kTileTokens - 1) * n) * g + kTileTokens * (kChainTiles - 1) * n) / (kTileTokens * kChainTiles) * b.n_kv_heads) + steps;
    const int64_t more = k > 0 ? k * chains_of(least, b.group) + (spare - k * (least - 1)) * ((g + kChainTiles - 1) / kChainTiles) / price : 0;
    const double priced = (double)((chains_of(b.max_q_len, b.group) + more) * b.n_kv_heads) + steps;
    by_tokens = padded > by_tokens ? padded : by_tokens;
    by_chunks = priced > by_chunks ? priced : by_chunks;
  }
  return (int64_t)((by_tokens < by_chunks ? by_tokens : by_chunks) + 0.5);
}

// Hybrid batches in workgroups of eight waves (attn_paged_kernel<D, true>): whether, and in how many.
// They pay where the batch waits for its chains.  us, workgroups of four waves and of eight, 28 / 4 heads of 128 if not said:
//   more places than two rounds of the chip keep its units full either way, and two chains share a unit better than one has it: 96
//   decode steps of 128 .. 1800 tokens and 4 chunks of 512 (648 places) 55.7 and 58.4, 16 chunks of 512 (1792) 55.4 and 68.2, 16 steps and
//   2 chunks of 300 with 32 / 32 heads (480) 28.5 and 30.3; but 4 chunks of 512 alone (456) 48.5 and 40.0, 23 of 61 .. 619 and 3 of 428
//   (352) 34.1 and 27.6, 55 of 171 .. 1712 and 4 of 308 (406) 32.8 and 32.2;
//   where contexts are far longer than the chunks, decode steps are what it waits for: 36 of 246 .. 2466 and 3 of 352 34.6 and
//   36.7, 59 of 51 .. 512 and one of 104 9.4 and 10.1, 63 of 42 .. 423 and 3 of 62 11.2 and 11.6, 30 of 113 .. 1138 and 3 of 168 16.4 and 16.9;
//   with a unit for every place from longer ones on: 25 of 114 .. 1142 and 4 of 102 13.3 and 12.0, 6 of 49 .. 492 and 2 of 97 9.5 and 8.4,
//   42 of 72 .. 723 and 4 of 64 11.9 and 12.2; whatever they are where chains are most of the places: a chunk of 512 behind 1536
//   keys 41.6 and 30.3;
//   shares of split contexts are not ranked, and two to a workgroup can be two long ones: 20 of 240 .. 2408 and 4 of 68 17.0 and 20.7;
//   with more decode steps than units the contexts decide, which the host does not see: 55 mixes of 60 .. 96 steps of up to 500 .. 1300 tokens and
//   1 .. 4 chunks of 120 .. 420 that pass take 0.92 of the time on average, between 0.68 and 1.09.
// The lengths are on the device.  Where the tokens are those of whole chunks of max_q_len beside decode steps of one token, to the
// token, that is what the batch is taken for: it is what a scheduler with a chunk size makes, and others hit it one time in
// max_q_len - 1.  (Then what the grid has no place for is done all the same, slower.)
// Any other batch may have far more chains than its tokens make at first sight, with 28 / 4 heads two per KV head for every request of 5 to 18
// new tokens (a draft that is verified), so there it is the most places that count, the grid has them all, and decode steps are ordered,
// one to a workgroup while there are units.  us with four waves, with eight by the look of the tokens, and now, requests of k tokens behind 300 .. 1100 keys and a
// chunk: 99 of 5 and 300 (864 chains) 46, 86 and 46, 63 of 6 and 256 (560) 31.5, 47 and 31.5, 40 of 8 and 300 (392) 26.7, 41.5 and 26.7, 20 of 8 and 256
// (164) 25.4, 25.4 and 25.4; chunks of 200, 100, 50, 25, 12 and 6 tokens alone 17.5, 14.0 and 14.0, one of 512 and six of 64 18.5, 14.8 and 14.8.
// The price: batches that may have more places than they do, as a chunk of 512, three of 40 and 40 decode steps 25.9, 18.3 and 25.9.
//   Beyond a unit for every place, four and eight waves with all places in the grid: up to 350 places 0.79 to 1.005 of the time; above
//   0.8 to 1.1, 20 chunks of 33 tokens and one of 400 (412) 17.9 and 19.8, 19 of 5 and 2 of 423 (376) 25.4 and 27.3; under tables of few
//   keys, where it is the start that counts, 30 of 5 behind up to 238 keys and 3 of 68 (316) 10.7 and 13.1, and with a unit for
//   every place 4 of 3 behind 112 and one of 34 6.1 and 6.7, 12 of 6 .. 139 and one of 108 7.2 and 7.3.
struct WideGrid {
  bool use;
  bool by_context;  // the decode steps are ordered whatever their contexts are
  int64_t workgroups;
};
inline WideGrid wide_grid(const Hybrid& b) {
  WideGrid g = {false, false, 0};
  const int64_t tokens = (int64_t)b.total_q - b.batch, chunk = b.max_q_len - 1;  // of chunks, beyond one for every request
  // (fewer tokens than that: max_q_len is a loose bound, and nothing is known of the chunks)
  if (b.batch > kWideMost || chunk < 1 || tokens < chunk) return g;
  const int64_t steps = (int64_t)b.batch * b.n_kv_heads * b.n_splits, longest = chains_of(b.max_q_len, b.group) * b.n_kv_heads;
  if (tokens % chunk == 0) {
    const int64_t chains = longest * (tokens / chunk), paired = (steps + 1) / 2;
    const bool all_at_once = steps + chains <= kUnits;
    g.use = (all_at_once || b.n_splits == 1 || steps <= chains) && paired + chains <= 470 && (steps * 2 <= chains || b.table_keys * 10 <= tokens * (all_at_once ? 28 : 20));
    // (find_work rounds two numbers of places up to multiples of 8)
    g.workgroups = paired + chains + chains / 4 + 16 + kTrailing;
    if (g.workgroups < kUnits + 16) g.workgroups = kUnits + 16;
    return g;
  }
  const bool all_at_once = places_most(b, b.n_splits) <= kUnits;
  const int64_t places = places_most(b, all_at_once ? b.n_splits : 0.5 * b.n_splits);
  g.by_context = true;
  g.use = (all_at_once ? b.table_keys >= 192 : places <= 350 && b.table_keys >= 300 && (b.n_splits == 1 || steps * 2 <= longest * 3)) &&
          (steps * 2 <= longest || b.table_keys * 10 <= tokens * (all_at_once ? 28 : 20));
  g.workgroups = places + b.n_kv_heads * b.n_splits + 16 + kTrailing;
  if (!all_at_once && g.workgroups < kUnits + 16) g.workgroups = kUnits + 16;
  return g;
}

}  // namespace rules
}  // namespace hydra
