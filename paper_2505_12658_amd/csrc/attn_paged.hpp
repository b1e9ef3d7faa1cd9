// Attention of a hybrid batch over the paged KV cache (gfx950).
//
// The paper's batch scheduler (Algorithm 1) fills one batch, under a token budget, with the decode
// requests (one new token each) and with chunks of prefill requests (get_chunked_size new tokens
// each); all of them attend to their request's KV cache, which is paged (Section 4.5; block size 16 in Section 5.1).
// Request b brings q_len new tokens and has kv_len tokens of context in the cache, the new ones
// included (written beforehand by the paged KV write).  New token i sees keys 0 .. kv_len - q_len + i:
// the causal mask aligned to the END of the context.  q_len == kv_len is an ordinary prefill,
// q_len == 1 a decode step.
//
// Decomposition: a workgroup of 4 waves takes up to four consecutive wave tiles of one (request, KV
// head); a wave tile is 32 new tokens of one query head, flattened as f = token_tile * group +
// head_in_group, so with grouped queries the waves share every K/V tile.  In the plain form K/V tiles of
// 64 keys are gathered row by row from the pages (a lane looks its row's page up in the block table, then
// the 16-byte pieces travel global -> LDS with direct-to-LDS loads) into two stages: tile t + 1 is
// fetched while tile t is used.  Scores are kept transposed (S^T = K Q^T, O^T += V^T P^T, as in the
// packed kernel) and the softmax is the textbook online one: running maximum and rescaling at every
// tile.  Two workgroups per compute unit.
// Requests with few new tokens (decode steps above all) take another form, in which the rows of ALL the query heads of
// a KV head share one tile and the four waves split the keys: attn_decode.hpp where there are at most 16 rows and the
// cache layout allows, run_packed_rows otherwise.
// When the batch is small for the chip or its contexts are long, the packed-rows form also splits a context
// over several workgroups and a second, small kernel merges their partial results (see n_splits).
// Groups of wave tiles run on the packed kernel's software pipeline where the cache layout allows (PagedSource);
// the loop at the end of attn_paged_kernel is the plain form of the same computation (no pipelining inside the
// wave, online softmax), which the other layouts and the groups that leave the pipeline's range take.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_decode.hpp"
#include "attn_fwd.hpp"
#include "attn_tiles.hpp"
#include "paged_args.hpp"

namespace hydra {
namespace paged {

constexpr int kPagedWavesPerSimd = 2;  // that attn_paged_kernel is built for

template <int D>
struct StageGeom : RowGeom<D> {
  using RowGeom<D>::kTileBytes;
  using RowGeom<D>::kPvChunks;
  static constexpr int kStageBytes = 2 * kTileBytes;  // K then V
  // A wave's slot in the packed-rows form: a stage of a HALF tile (32 keys of K, then of V) during the loop,
  // its unnormalised output (kPvChunks * 16 registers x 64 lanes x 4 bytes) for the merge.  Four slots; the
  // wave-tile form uses the same memory as its two 64-key stages.
  static constexpr int kHalfStageBytes = kStageBytes / 2;
  static constexpr int kPartialBytes = kPvChunks * 16 * 64 * 4;
  static constexpr int kSlotBytes = kHalfStageBytes > kPartialBytes ? kHalfStageBytes : kPartialBytes;
  static constexpr int kLdsBytes = (4 * kSlotBytes > 2 * kStageBytes ? 4 * kSlotBytes : 2 * kStageBytes) + 64;  // slack: D=80 reads V columns 80..95
};

#if defined(__HIP_DEVICE_COMPILE__)
// The K/V tiles are gathered from the pages in two moves, so that the block-table lookup of a tile is in
// flight while the tile before it is fetched and used (done in one move, every tile would pay the lookup's
// round trip before its loads can even be issued):
//   fetch_tile_slots: per load instruction of this wave, the cache row ("slot" = block * block_size + offset)
//     of this lane's key.  Load instructions first, first + step, ... (a workgroup's four waves share a tile
//     with first = wave, step = 4; a wave that owns a whole tile uses first = 0, step = 1).  Keys past the end
//     of the context re-read the last valid key (always masked later).  Block ids are clamped to the cache,
//     so a corrupt table cannot make the loads leave it.
//   issue_tile_loads: the direct-to-LDS loads of the K rows and V rows of those slots (KEYS keys: 64, or 32
//     for a half tile; K rows first, then V rows).
template <int D, int KEYS, int STEP>
struct TileSlots {
  static constexpr int kLoadInstr = KEYS * StageGeom<D>::kRowBytes / 1024;
  static constexpr int kCount = (kLoadInstr + STEP - 1) / STEP;
  int32_t slot[kCount];  // (the host refuses caches of 2^31 rows or more)
};

// (in two steps for callers that keep other loads in flight across the look-up: the table entries are requested
// by request_tile_blocks and only touched, which is what the compiler waits for, by slots_from_blocks)
template <int D, int KEYS, int STEP>
__device__ __forceinline__ void request_tile_blocks(TileSlots<D, KEYS, STEP>& ts, const PagedArgs& a, const int32_t* table, int first, int lane,
                                                    int kv_len, int kv0) {
  using G = StageGeom<D>;
#pragma unroll
  for (int u = 0; u < TileSlots<D, KEYS, STEP>::kCount; ++u) {
    const int instr = first + STEP * u;
    const int row = (instr * 64 + lane) / G::kChunks;
    int tok = kv0 + row;
    tok = tok < kv_len ? tok : kv_len - 1;
    ts.slot[u] = table[tok >> a.block_shift];
  }
}
template <int D, int KEYS, int STEP>
__device__ __forceinline__ void slots_from_blocks(TileSlots<D, KEYS, STEP>& ts, const PagedArgs& a, int first, int lane, int kv_len, int kv0) {
  using G = StageGeom<D>;
  const int in_block = (1 << a.block_shift) - 1;
#pragma unroll
  for (int u = 0; u < TileSlots<D, KEYS, STEP>::kCount; ++u) {
    const int instr = first + STEP * u;
    const int row = (instr * 64 + lane) / G::kChunks;
    int tok = kv0 + row;
    tok = tok < kv_len ? tok : kv_len - 1;
    int block = ts.slot[u];
    block = block < 0 ? 0 : (block >= a.num_blocks ? a.num_blocks - 1 : block);
    ts.slot[u] = (block << a.block_shift) + (tok & in_block);
  }
}
template <int D, int KEYS, int STEP>
__device__ __forceinline__ void fetch_tile_slots(TileSlots<D, KEYS, STEP>& ts, const PagedArgs& a, const int32_t* table, int first, int lane,
                                                 int kv_len, int kv0) {
  request_tile_blocks(ts, a, table, first, lane, kv_len, kv0);
  slots_from_blocks(ts, a, first, lane, kv_len, kv0);
}

// CPOL: cache-policy bits of the load instructions (2 = nt: lines marked for early replacement, for rows that no
// other workgroup reads again).
template <int CPOL = 0, int D, int KEYS, int STEP>
__device__ __forceinline__ void issue_tile_loads(const TileSlots<D, KEYS, STEP>& ts, const PagedArgs& a, unsigned char* stage, int first, int lane,
                                                 int kv_head) {
  using G = StageGeom<D>;
  constexpr int kTileBytes = KEYS * G::kRowBytes;
  const int64_t row_elems = (int64_t)a.n_kv_heads * D;
#pragma unroll
  for (int u = 0; u < TileSlots<D, KEYS, STEP>::kCount; ++u) {
    const int instr = first + STEP * u;
    if (instr < TileSlots<D, KEYS, STEP>::kLoadInstr) {
      const int flat = instr * 64 + lane;
      const int row = flat / G::kChunks;
      const int phys = flat % G::kChunks;
      const uint16_t* kp = a.k_cache + ts.slot[u] * row_elems + kv_head * D + k_swizzle<D>(row, phys) * 8;
      const uint16_t* vp = a.v_cache + ts.slot[u] * row_elems + kv_head * D + v_swizzle<D>(row, phys) * 8;
      __builtin_amdgcn_global_load_lds(HYDRA_GLOBAL_PTR(kp), HYDRA_LDS_PTR(stage + instr * 1024), 16, 0, CPOL);
      __builtin_amdgcn_global_load_lds(HYDRA_GLOBAL_PTR(vp), HYDRA_LDS_PTR(stage + kTileBytes + instr * 1024), 16, 0, CPOL);
    }
  }
}

// ---- the wave-tile form on the packed kernel's pipeline --------------------------------------------------
// A prefill chunk is causal attention whose queries are the LAST q_len positions of a context of kv_len keys,
// so a group of four wave tiles runs through the packed kernel's item loop (attn_fwd.hpp: software-pipelined
// key-block steps, fixed softmax reference with a row-sum check) with this source: one item, its K/V tiles
// gathered from the pages.
//
// The gatherer relies on a load instruction's rows (1024 bytes: 4 rows at head_dim 128, 8 at 64) lying in ONE
// cache block, which holds when the block size is at least that many rows (tiles start at multiples of 64 keys):
// the block is then the same for all lanes, the load goes through a buffer descriptor that starts at the group's
// first row and ends with its last valid row (rows past the end of the context arrive as zeros, as in the packed
// kernel), and a tile needs one table entry per load instruction of the wave.  Those entries are looked up one
// tile ahead: lane u of the wave fetches the entry of the wave's load u, the iteration-end wait for all loads
// covers it, and the next iteration's issue reads it lane by lane into scalar registers.  The V tile of an
// iteration comes from the blocks its K tile came from one iteration earlier, so they are kept.
// head_dim 80 (a row is not a whole fraction of 1024 bytes) and smaller blocks take the plain loop further down.
// LOADERS: waves that do nothing but load tiles (see attn_item_loop).
template <int LOADERS = 0>
struct PagedSource {
  static constexpr bool kPaged = true, kOneItem = true;
  static constexpr int kTeams = 1, kTiles = kWavesPerItem;
  static constexpr int kLoaders = LOADERS, kStageRows = LOADERS > 0 ? kWavesPerItem * kWaveTileRows : 0;
  template <int D>
  static constexpr int kWavesPerSimd = kPagedWavesPerSimd;
  const PagedArgs* args;
  const int32_t* table;  // the request's row of the block table
  int64_t q_start;       // first new token of the request in the packed q / out
  int q_len, kv_len;     // new tokens, context (new tokens included)
  int f0, kv_head;       // first flattened wave tile of the group, KV head

  template <int D>
  struct Gather {
    using G = TileGeom<D>;
    static constexpr int kPerWave = G::kLoadInstr / 4;          // load instructions per wave and tile
    static constexpr int kRowsPerInstr = 1024 / G::kRowBytes;   // rows one load instruction covers
    static_assert(G::kLoadInstr % 4 == 0 && 1024 % G::kRowBytes == 0 && TileLoader<D>::kUniformStep, "whole rows per instruction");
    uint32_t k_lo, k_hi, v_lo, v_hi;  // byte address of this KV head's part of cache row 0 (uniform)
    uint32_t row_bytes;               // bytes between cache rows (uniform)
    uint32_t k_lane_off, v_lane_off;  // this lane's 16 bytes inside a load instruction's rows
    const int32_t* table;
    int kv_len, block_shift, last_block, last_entry, wave;
    int next_tile;              // the next K tile to issue, whose table entries `pending` holds
    int32_t pending;            // lane u < kPerWave: table entry of this wave's load u of tile next_tile
    int32_t v_block[kPerWave];  // blocks of the next V tile to issue (uniform)

    // (first key of the rows of this wave's load u of a tile)
    __device__ __forceinline__ int first_key(int tile, int u) const { return tile * kKvTileRows + kRowsPerInstr * (wave + 4 * u); }

    __device__ __forceinline__ void lookup(int tile) {
      // (the lane number is formed here, two instructions, instead of living in a register through the hot loop)
      const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
      pending = 0;
      if (lane < kPerWave) {
        int entry = first_key(tile, lane) >> block_shift;
        entry = entry < last_entry ? entry : last_entry;  // (tiles past the context are looked up but never loaded)
        pending = table[entry];
      }
    }
    __device__ __forceinline__ void take(int32_t (&block)[kPerWave]) const {
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) {
        const int b = __builtin_amdgcn_readlane(pending, u);
        block[u] = b < 0 ? 0 : (b > last_block ? last_block : b);  // a corrupt table cannot make the loads leave the cache
      }
    }
    __device__ __forceinline__ void issue_tile(int tile, const int32_t (&block)[kPerWave], uint32_t lo, uint32_t hi, uint32_t lane_off,
                                               uint32_t lds_dst) const {
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) {
        const int key = first_key(tile, u);
        const uint32_t slot = ((uint32_t)block[u] << block_shift) + ((uint32_t)key & ((1u << block_shift) - 1u));
        const uint64_t base = (((uint64_t)hi << 32) | lo) + (uint64_t)slot * row_bytes;
        int valid = kv_len - key;
        valid = valid > kRowsPerInstr ? kRowsPerInstr : valid;
        u32x4_t rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
        rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
        rsrc[2] = __builtin_amdgcn_readfirstlane(valid > 0 ? (uint32_t)(valid - 1) * row_bytes + D * 2 : 0u);
        rsrc[3] = 0x00020000u;
        const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst + (wave + 4 * u) * 1024);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(m0), "v"(lane_off), "s"(rsrc));
      }
    }

    __device__ __forceinline__ void init(const PagedSource& src, int kv_head, int wave_, int lane) {
      const PagedArgs& a = *src.args;
      wave = wave_;
      __builtin_assume(wave >= 0 && wave < kWavesPerItem);
      table = src.table;
      kv_len = src.kv_len;
      block_shift = a.block_shift;
      last_block = a.num_blocks - 1;
      last_entry = a.max_blocks_per_seq - 1;
      row_bytes = __builtin_amdgcn_readfirstlane((uint32_t)a.n_kv_heads * (D * 2));
      const uint64_t kb = (uint64_t)(uintptr_t)(a.k_cache + (int64_t)kv_head * D), vb = (uint64_t)(uintptr_t)(a.v_cache + (int64_t)kv_head * D);
      k_lo = __builtin_amdgcn_readfirstlane((uint32_t)kb);
      k_hi = __builtin_amdgcn_readfirstlane((uint32_t)(kb >> 32));
      v_lo = __builtin_amdgcn_readfirstlane((uint32_t)vb);
      v_hi = __builtin_amdgcn_readfirstlane((uint32_t)(vb >> 32));
      // (the swizzles repeat from one load instruction of the wave to its next, 16 or 32 rows further on)
      const int in_instr = lane / G::kChunks, phys = lane % G::kChunks, row = kRowsPerInstr * wave + in_instr;
      k_lane_off = (uint32_t)in_instr * row_bytes + k_swizzle<D>(row, phys) * 16;
      v_lane_off = (uint32_t)in_instr * row_bytes + v_swizzle<D>(row, phys) * 16;
      next_tile = 0;
      lookup(0);
    }
    // K tile 0
    __device__ __forceinline__ void issue_first(uint32_t k_dst) {
      take(v_block);
      issue_tile(0, v_block, k_lo, k_hi, k_lane_off, k_dst);
      next_tile = 1;
      lookup(1);
    }
    // The V tile that goes with the K tile issued last (if has_v) and the next K tile (if has_k).  Both sets of
    // table entries are in scalar registers before the first load goes out: the compiler waits for the look-up
    // where its result is first read, and a wait placed behind tile loads would wait for those as well.
    __device__ __forceinline__ void issue(bool has_v, uint32_t v_dst, bool has_k, uint32_t k_dst) {
      if (!has_v && !has_k) return;
      int32_t k_block[kPerWave];
      take(k_block);
      if (has_v) issue_tile(next_tile - 1, v_block, v_lo, v_hi, v_lane_off, v_dst);
      if (has_k) issue_tile(next_tile, k_block, k_lo, k_hi, k_lane_off, k_dst);
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) v_block[u] = k_block[u];
      ++next_tile;
      lookup(next_tile);
    }
  };

  // One of WAVES waves that load the K tiles, or the V tiles, of the item one after the other.
  template <int D, int WAVES>
  struct Loader {
    using G = TileGeom<D>;
    static constexpr int kPerWave = G::kLoadInstr / WAVES;
    static constexpr int kRowsPerInstr = 1024 / G::kRowBytes;
    static constexpr int kPeriod = kRowsPerInstr * WAVES % 16 == 0 ? 1 : 2;  // loads after which the swizzles repeat
    static_assert(G::kLoadInstr % WAVES == 0 && 1024 % G::kRowBytes == 0 && kRowsPerInstr * WAVES * kPeriod % 16 == 0 && kPerWave <= 64, "whole rows per instruction");
    uint32_t lo, hi;             // byte address of this KV head's part of cache row 0 (uniform)
    uint32_t row_bytes;          // bytes between cache rows (uniform)
    uint32_t lane_off[kPeriod];  // this lane's 16 bytes inside a load instruction's rows
    const int32_t* table;
    int kv_len, block_shift, last_block, last_entry, number, lane;
    int next_tile;    // the next tile to issue, whose table entries `pending` holds
    int32_t pending;  // lane u < kPerWave: table entry of this wave's load u of tile next_tile

    __device__ __forceinline__ int first_key(int tile, int u) const { return tile * kKvTileRows + kRowsPerInstr * (number + WAVES * u); }
    __device__ __forceinline__ void lookup(int tile) {
      pending = 0;
      if (lane < kPerWave) {
        int entry = first_key(tile, lane) >> block_shift;
        entry = entry < last_entry ? entry : last_entry;  // (tiles past the context are looked up but never loaded)
        pending = table[entry];
      }
    }
    __device__ __forceinline__ void init(const PagedSource& src, bool is_v, int kv_head, int number_, int lane_) {
      const PagedArgs& a = *src.args;
      number = number_;
      lane = lane_;
      table = src.table;
      kv_len = src.kv_len;
      block_shift = a.block_shift;
      last_block = a.num_blocks - 1;
      last_entry = a.max_blocks_per_seq - 1;
      row_bytes = __builtin_amdgcn_readfirstlane((uint32_t)a.n_kv_heads * (D * 2));
      const uint64_t base = (uint64_t)(uintptr_t)((is_v ? a.v_cache : a.k_cache) + (int64_t)kv_head * D);
      lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
      hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
      const int in_instr = lane / G::kChunks, phys = lane % G::kChunks;
#pragma unroll
      for (int u = 0; u < kPeriod; ++u) {
        const int row = kRowsPerInstr * (number + WAVES * u) + in_instr;
        lane_off[u] = (uint32_t)in_instr * row_bytes + (is_v ? v_swizzle<D>(row, phys) : k_swizzle<D>(row, phys)) * 16;
      }
      next_tile = 0;
      lookup(0);
    }
    __device__ __forceinline__ void issue_next(uint32_t lds_dst) {
      int32_t block[kPerWave];  // (all in scalar registers before the first load goes out, see Gather::issue)
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) {
        const int b = __builtin_amdgcn_readlane(pending, u);
        block[u] = b < 0 ? 0 : (b > last_block ? last_block : b);  // a corrupt table cannot make the loads leave the cache
      }
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) {
        const int key = first_key(next_tile, u);
        const uint32_t slot = ((uint32_t)block[u] << block_shift) + ((uint32_t)key & ((1u << block_shift) - 1u));
        const uint64_t base = (((uint64_t)hi << 32) | lo) + (uint64_t)slot * row_bytes;
        int valid = kv_len - key;
        valid = valid > kRowsPerInstr ? kRowsPerInstr : valid;
        u32x4_t rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
        rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
        rsrc[2] = __builtin_amdgcn_readfirstlane(valid > 0 ? (uint32_t)(valid - 1) * row_bytes + D * 2 : 0u);
        rsrc[3] = 0x00020000u;
        const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst + (number + WAVES * u) * 1024);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(m0), "v"(lane_off[u % kPeriod]), "s"(rsrc));
      }
      ++next_tile;
      lookup(next_tile);
    }
  };
};

// The same rows on their way through registers: ordinary loads, which complete in the order they were issued and
// can be counted, so that a wave can have the NEXT tile's rows in flight while it computes on the current one
// (direct-to-LDS loads land in no particular order: a wave that uses them can only wait for all of its loads).
// The rows are written to the stage, in the layout the direct loads would have produced, when their turn comes.
template <int D, int KEYS>
struct TileRegs {
  static constexpr int kLoadInstr = KEYS * StageGeom<D>::kRowBytes / 1024;
  u32x4_t k[kLoadInstr], v[kLoadInstr];
};
template <int D, int KEYS>
__device__ __forceinline__ void load_tile_regs(TileRegs<D, KEYS>& regs, const TileSlots<D, KEYS, 1>& ts, const PagedArgs& a, int lane, int kv_head) {
  using G = StageGeom<D>;
  const int64_t row_elems = (int64_t)a.n_kv_heads * D;
#pragma unroll
  for (int u = 0; u < TileRegs<D, KEYS>::kLoadInstr; ++u) {
    const int flat = u * 64 + lane;
    const int row = flat / G::kChunks, phys = flat % G::kChunks;
    const uint16_t* kp = a.k_cache + ts.slot[u] * row_elems + kv_head * D + k_swizzle<D>(row, phys) * 8;
    const uint16_t* vp = a.v_cache + ts.slot[u] * row_elems + kv_head * D + v_swizzle<D>(row, phys) * 8;
    // (nt: each key of the context is read by exactly one wave of one workgroup)
    regs.k[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(kp));
    regs.v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(vp));
  }
}
template <int D, int KEYS>
__device__ __forceinline__ void store_tile_regs(const TileRegs<D, KEYS>& regs, unsigned char* stage, int lane) {
  constexpr int kTileBytes = KEYS * StageGeom<D>::kRowBytes;
#pragma unroll
  for (int u = 0; u < TileRegs<D, KEYS>::kLoadInstr; ++u) {
    *reinterpret_cast<u32x4_t*>(stage + u * 1024 + lane * 16) = regs.k[u];
    *reinterpret_cast<u32x4_t*>(stage + kTileBytes + u * 1024 + lane * 16) = regs.v[u];
  }
}

// A wave's state for 32 * QS query rows (QS sub-tiles of 32) and the arithmetic of one 64-key tile:
// S^T = K Q^T, mask, online softmax (running maximum, rescaling), O^T += V^T P^T.
template <int D, int QS>
struct WaveTile {
  using G = StageGeom<D>;
  static constexpr int KS = G::kQkSteps;
  static constexpr int CC = G::kPvChunks;
  static constexpr int ROWB = G::kRowBytes;
  bf16x8_t qf[QS][KS];  // B operand: lane (m, hf) holds its row's columns hf*D/2 + 8*s .. +7
  int q_lim[QS];        // largest visible key index of this lane's row in sub-tile qs
  uint32_t k_off[KS], v_off[CC];
  f32x16_t o_acc[QS][CC];
  float row_max[QS], row_sum[QS];
  float c;  // softmax_scale * log2(e)
  int hf;

  __device__ __forceinline__ void init(int lane, float scale_log2) {
    const int m = lane & 31, sl = lane & 15, grp = (lane >> 4) & 1;
    hf = lane >> 5;
    c = scale_log2;
#pragma unroll
    for (int s = 0; s < KS; ++s) k_off[s] = m * ROWB + k_swizzle<D>(m, KS * hf + s) * 16;
    const int r = 4 * hf + (sl >> 2);
#pragma unroll
    for (int cc = 0; cc < CC; ++cc) {
      const int chunk = 4 * cc + 2 * grp + ((sl & 3) >> 1);
      v_off[cc] = r * ROWB + v_swizzle<D>(r, chunk) * 16 + 8 * (sl & 1);  // inside the V rows of a stage
    }
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      row_max[qs] = kLowest;
      row_sum[qs] = 0.f;
#pragma unroll
      for (int cc = 0; cc < CC; ++cc)
#pragma unroll
        for (int r2 = 0; r2 < 16; ++r2) o_acc[qs][cc][r2] = 0.f;
    }
  }
  // row pointer: this lane's query row of sub-tile qs (columns 0 .. D-1 contiguous)
  __device__ __forceinline__ void load_q(int qs, const uint16_t* row_ptr, int limit) {
    q_lim[qs] = limit;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[qs][s] = *reinterpret_cast<const bf16x8_t*>(row_ptr + hf * (D / 2) + 8 * s);
  }

  // one K/V tile of 32 * RBN keys whose first key is kv0, already complete in `stage` (K rows, then V rows);
  // need_mask: some key of the tile lies past some row's limit
  template <int RBN = 2>
  __device__ __forceinline__ void tile(const unsigned char* stage, int kv0, bool need_mask) {
    // ---- S^T = K Q^T ----
    f32x16_t s_acc[RBN][QS];  // [rb][qs]
    // (consecutive matrix instructions go to different accumulators wherever there are several: one that
    // continues the accumulator of the instruction right before it waits for that one to finish)
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
      for (int qs = 0; qs < QS; ++qs)
#pragma unroll
        for (int r = 0; r < 16; ++r) s_acc[rb][qs][r] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb) {
        const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(stage + rb * 32 * ROWB + k_off[s]);
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) s_acc[rb][qs] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qs][s], s_acc[rb][qs], 0, 0, 0);
      }
    if (need_mask) {
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kv0 + 32 * rb + 8 * (r >> 2) + 4 * hf + (r & 3);
#pragma unroll
          for (int qs = 0; qs < QS; ++qs)
            if (key > q_lim[qs]) s_acc[rb][qs][r] = -__builtin_inff();
        }
    }
    // ---- online softmax, P in bf16 ----
    bf16x8_t p_frag[QS][RBN][2];  // [qs][rb][s2]
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      float tmax = s_acc[0][qs][0];
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s_acc[rb][qs][r]);
      tmax = max_with_other_half(tmax);
      // (a row whose keys are all masked so far keeps the initial, very negative maximum: every
      // exponential below is then exp2(-inf) = 0)
      const float m_new = fmaxf(row_max[qs], tmax);
      const float alpha = fast_exp2((row_max[qs] - m_new) * c);
      row_max[qs] = m_new;
      const float mc = reference_exponent(m_new, c);
      float psum = 0.f;
#pragma unroll
      for (int rb = 0; rb < RBN; ++rb) {
        float p[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = fast_exp2(__builtin_fmaf(s_acc[rb][qs][r], c, -mc));
        if (need_mask) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = kv0 + 32 * rb + 8 * (r >> 2) + 4 * hf + (r & 3);
            if (key > q_lim[qs]) p[r] = 0.f;
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) psum += p[r];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            f32x2_t pr = {p[8 * s2 + e], p[8 * s2 + e + 1]};
            bf16x2_t pb = __builtin_convertvector(pr, bf16x2_t);
            p_frag[qs][rb][s2][e] = pb[0];
            p_frag[qs][rb][s2][e + 1] = pb[1];
          }
      }
      row_sum[qs] = row_sum[qs] * alpha + psum;
#pragma unroll
      for (int cc = 0; cc < CC; ++cc)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[qs][cc][r] *= alpha;
    }
    // ---- O^T += V^T P^T ----
#pragma unroll
    for (int rb = 0; rb < RBN; ++rb)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int cc = 0; cc < CC; ++cc) {
          const unsigned char* vp = stage + RBN * 32 * ROWB + v_off[cc] + (32 * rb + 16 * s2) * ROWB;
          const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)HYDRA_LDS_PTR(vp));
          const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)HYDRA_LDS_PTR(vp + 8 * ROWB));
          typedef __attribute__((ext_vector_type(8))) short s16x8_t;
          const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          const bf16x8_t vf = __builtin_bit_cast(bf16x8_t, both);
#pragma unroll
          for (int qs = 0; qs < QS; ++qs) o_acc[qs][cc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p_frag[qs][rb][s2], o_acc[qs][cc], 0, 0, 0);
        }
  }

  // normalise this lane's row of sub-tile qs, round to bf16 and store it at out_row (D contiguous elements)
  __device__ __forceinline__ void store_row(int qs, uint16_t* out_row) {
    const float total = sum_with_other_half(row_sum[qs]);
    const float inv = 1.0f / total;
    if (out_row == nullptr) return;  // (every lane takes part in the exchange above)
#pragma unroll
    for (int cc = 0; cc < CC; ++cc)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int col = 32 * cc + 8 * g4 + 4 * hf;
        if (col < D) {
          f32x2_t a0 = {o_acc[qs][cc][4 * g4] * inv, o_acc[qs][cc][4 * g4 + 1] * inv};
          f32x2_t a1 = {o_acc[qs][cc][4 * g4 + 2] * inv, o_acc[qs][cc][4 * g4 + 3] * inv};
          const bf16x2_t b0 = __builtin_convertvector(a0, bf16x2_t);
          const bf16x2_t b1 = __builtin_convertvector(a1, bf16x2_t);
          u32x2_t pk = {__builtin_bit_cast(uint32_t, b0), __builtin_bit_cast(uint32_t, b1)};
          *reinterpret_cast<u32x2_t*>(out_row + col) = pk;
        }
      }
  }
};

// Few new tokens (q_len * group <= 32: decode steps above all): ALL (token, head) pairs of one (request, KV
// head) form one tile of rows, row = token * group + head_in_group, and the four waves split the KEYS
// instead of the rows: wave w takes the half tiles (32 keys) w, w + 4, ... into a stage of its own (no
// workgroup barrier inside the loop; a wave's next half tile travels through registers while it computes on
// the current one, see TileRegs), and the four partial results (maximum, sum, unnormalised output per row)
// are merged through LDS at the end.
// thread, result: see run_decode.
template <int D>
__device__ __forceinline__ bool run_packed_rows(const PagedArgs& a, unsigned char* smem, float* s_stats, const int32_t* table, int64_t q_start,
                                                int q_len, int kv_len, int kv_head, int request, int split, int thread) {
  using G = StageGeom<D>;
  using W = WaveTile<D, 1>;
  constexpr int kHalfKeys = kKvTileRows / 2;
  const int lane = thread & 63;
  const int wave = __builtin_amdgcn_readfirstlane(thread >> 6);
  const int m = lane & 31;
  const int shift = kv_len - q_len;
  const int n_rows = q_len * a.group;

  W w;
  w.init(lane, a.scale_log2);
  int r = m;
  const bool valid = r < n_rows;
  r = valid ? r : n_rows - 1;
  const int token = quotient(r, a.group);
  const int head = kv_head * a.group + (r - token * a.group);
  w.load_q(0, a.q + (q_start + token) * a.q_stride + head * D, shift + token);

  unsigned char* stage = smem + wave * G::kSlotBytes;
  const int n_halves = (kv_len + kHalfKeys - 1) / kHalfKeys;
  int h_begin, h_end;
  int per_share, n_shares;
  share_plan(n_halves, a.n_splits, a.least_log2, per_share, n_shares);
  split_range(n_halves, per_share, split, h_begin, h_end);
  if (h_begin >= h_end) return false;  // past the context's last share: the combine kernel knows and skips it
  const bool whole = n_shares == 1;  // the context is one share: this workgroup writes the output
  // The rows of half tile h + 4 travel (into registers) while half tile h is computed on, and the block-table
  // look-up of half tile h + 8 travels behind them; its entries are not touched before the top of the next round.
  TileSlots<D, kHalfKeys, 1> slots;
  TileRegs<D, kHalfKeys> regs;
  if (h_begin + wave < h_end) {
    fetch_tile_slots(slots, a, table, 0, lane, kv_len, (h_begin + wave) * kHalfKeys);
    load_tile_regs(regs, slots, a, lane, kv_head);
    if (h_begin + wave + kWavesPerGroup < h_end) request_tile_blocks(slots, a, table, 0, lane, kv_len, (h_begin + wave + kWavesPerGroup) * kHalfKeys);
  }
  for (int h = h_begin + wave; h < h_end; h += kWavesPerGroup) {
    const int kv0 = h * kHalfKeys;
    store_tile_regs(regs, stage, lane);
    if (h + kWavesPerGroup < h_end) {
      slots_from_blocks(slots, a, 0, lane, kv_len, (h + kWavesPerGroup) * kHalfKeys);
      load_tile_regs(regs, slots, a, lane, kv_head);
      if (h + 2 * kWavesPerGroup < h_end) request_tile_blocks(slots, a, table, 0, lane, kv_len, (h + 2 * kWavesPerGroup) * kHalfKeys);
    }
    __builtin_amdgcn_sched_barrier(0);  // (the loads go out before the arithmetic, not wherever the scheduler finds room)
    w.template tile<1>(stage, kv0, kv0 + kHalfKeys - 1 > shift);
  }

  // ---- merge the four waves' partial results ----
  // statistics: s_stats[wave * 64 + lane] = maximum, the sums 256 floats further on (the maximum is the same
  // in both lanes of a row, the sum is the lane's half)
  s_stats[wave * 64 + lane] = w.row_max[0];
  s_stats[256 + wave * 64 + lane] = w.row_sum[0];
  // unnormalised outputs, register by register, lane-major, into the wave's own slot
  float* mine = reinterpret_cast<float*>(stage);
#pragma unroll
  for (int cc = 0; cc < W::CC; ++cc)
#pragma unroll
    for (int i = 0; i < 16; ++i) mine[(cc * 16 + i) * 64 + lane] = w.o_acc[0][cc][i];
  __syncthreads();
  if (wave != 0) return true;
  float scale_of[kWavesPerGroup];
  {
    float top = s_stats[lane];
#pragma unroll
    for (int o = 1; o < kWavesPerGroup; ++o) top = fmaxf(top, s_stats[o * 64 + lane]);
    float total = 0.f;
#pragma unroll
    for (int o = 0; o < kWavesPerGroup; ++o) {
      // (a wave that saw no key of this row still holds the initial maximum: weight 0)
      scale_of[o] = fast_exp2((s_stats[o * 64 + lane] - top) * w.c);
      total += scale_of[o] * s_stats[256 + o * 64 + lane];
    }
    w.row_sum[0] = total;
  }
#pragma unroll
  for (int cc = 0; cc < W::CC; ++cc)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float acc = w.o_acc[0][cc][i] * scale_of[0];
#pragma unroll
      for (int o = 1; o < kWavesPerGroup; ++o)
        acc += scale_of[o] * reinterpret_cast<const float*>(smem + o * G::kSlotBytes)[(cc * 16 + i) * 64 + lane];
      w.o_acc[0][cc][i] = acc;
    }
  if (whole) {
    w.store_row(0, valid ? a.out + ((q_start + token) * a.n_q_heads + head) * D : nullptr);
    return true;
  }
  // this share's partial result: the row's maximum, its sum (both halves of the row added up) and its
  // unnormalised output, for the combine kernel
  const float total = sum_with_other_half(w.row_sum[0]);
  float top = s_stats[lane];
#pragma unroll
  for (int o = 1; o < kWavesPerGroup; ++o) top = fmaxf(top, s_stats[o * 64 + lane]);
  float* rec = a.partials + (((int64_t)request * a.n_kv_heads + kv_head) * a.n_splits + split) * kPartialFloats<D>;
  if (valid) {
    if (w.hf == 0) {
      rec[m] = top;
      rec[kRows + m] = total;
    }
    float* row = rec + 2 * kRows + m * D;
#pragma unroll
    for (int cc = 0; cc < W::CC; ++cc)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int col = 32 * cc + 8 * g4 + 4 * w.hf;
        if (col < D) {
          f32x4_t v = {w.o_acc[0][cc][4 * g4], w.o_acc[0][cc][4 * g4 + 1], w.o_acc[0][cc][4 * g4 + 2], w.o_acc[0][cc][4 * g4 + 3]};
          *reinterpret_cast<f32x4_t*>(row + col) = v;
        }
      }
  }
  return true;
}

#endif  // __HIP_DEVICE_COMPILE__

// One-dimensional grid of workgroups of two kinds:
//   - decode steps and chunks of a few tokens, in the decode form or the packed-rows form: n_splits workgroups per
//     (request, KV head), each a share of the context;
//   - prefill chunks, in the wave-tile form: a workgroup per group of four wave tiles and KV head.  The groups are counted
//     off with the longest context first and inside a request from the last token tile down (which sees the most keys);
//     neighbouring workgroups have the same group and the next KV head.
// The host sizes the grid from the total number of new tokens (it cannot see the lengths); workgroups past the last group
// leave at once.  Which work a workgroup has, it finds out for itself: find_work for batches of up to kOrderedMost requests;
// for larger ones decode steps have the first batch * n_kv_heads * n_splits workgroups in the order of the requests, and a
// chunk's workgroup finds its group by a scan over the requests in LDS (the 256 threads add up the groups of a slice of the
// requests each, and the requests that have groups are ranked by context).
// The hardware starts workgroups in index order.  Both kinds live in one kernel so that the decode requests and the prefill
// chunks of a batch run side by side on the chip; two workgroups per compute unit (a wave keeps within 256 registers, a
// workgroup within half of the LDS).
// Wide workgroups (512 threads, one to a compute unit) are for batches that wait for their chains: four waves compute a chain and
// four load its tiles (attn_item_loop), so that a key tile takes 0.8 us instead of 1.1 (of which a third was the issue of the loads and
// their latency behind it), 1.0 with the whole chip at work; two chains to a unit take 1.5 each, which is the better rate where
// there is enough to fill the chip.  A wide workgroup has one decode step (share, packed-rows request) as long as the chip has units for
// all places, else the shortest are second ones: the halves of its waves take one each.  us, four waves and eight, 28 / 4 heads of 128: a
// chunk of 512 tokens alone 13.8 and 11.4, behind 1536 keys 41.2 and 30.3; 4 chunks of 128 14.1 and 11.6; 24 decode steps of 91 .. 916 and
// 4 chunks of 158 17.1 and 14.4, 53 of 50 .. 508 and 4 of 286 28.4 and 22.7, 76 of 44 .. 441 and 4 of 72 14.7 and 12.1; the same bits
// (but for places that the grid does not have, see run_place).
constexpr int kFirstLayer = kUnits;  // workgroups i and i + 256 of a grid share a compute unit
constexpr int kLongChain = 8;        // key tiles from which on a chunk's workgroups are kept apart from the decode steps'
constexpr int kStepUnits = 128;      // compute units that the chains leave to the decode steps
constexpr int kFewChunks = 4;        // as many are ranked one by one
constexpr int kTrailing = 32;        // places at the end of a wide grid that are chains at least, if not all places fit the grid
constexpr float kChainKeysPerStep = 2 * 32 * 0.9f;  // keys of a chain that take as long as a step of both of a wide workgroup's decode steps

// Context up to which a hybrid batch keeps the order of its requests.  To order it costs every workgroup up to 2 us where the
// lengths fill REGS = 4 registers (129 to 256 requests), 0.5 where they fill two, 0.3 with one, paid once per round of workgroups;
// it saves a part of the longest context's time.  So the limit grows with the pairs, and is in keys of head_dim 128 (a key of 64 takes
// half as long).  us, the order of the batch and ordered, 28 / 4 heads of 128 if not said: 248 decode steps of 19 .. 194 tokens and
// a chunk of 21 14.9 and 16.0, 250 of 160 .. 320 and 3 of 167 33.3 and 38.3, 177 of 362 .. 724 and 3 of 59 36.7 and 35.1, 232 of 1151 ..
// 2303 and 2 of 24 133.6 and 122.4; 203 of 20 .. 204 and 8 of 34 with 16 heads of 64 29.3 and 37.1; 102 of 17 .. 112 and one of 60 7.3
// and 8.2, 88 of 108 .. 217 and 3 of 129 15.5 and 16.7, 84 of 49 .. 494 and one of 27 14.5 and 10.8, 95 of 125 .. 1253 and 3 of 22 29.6
// and 24.2, but 111 of 37 .. 375 and 4 of 111 17.5 and 19.0, 120 of 61 .. 615 and 4 of 100 21.2 and 23.4; 32 of 167 .. 334 and 10 of 40 with
// 16 / 8 heads of 80 12.6 and 14.5, 45 of 128 .. 1288 and 6 of 410 with 32 heads 97.1 and 90.2.
// Without chunks it costs less, and a batch of no more pairs than compute units gains nothing: 3 requests of 17 new tokens behind up to 189
// keys, 16 heads of 64 under a table of 8192, 6.4 and 6.8; 97 of 3 behind 18 .. 176, 28 / 4 heads of 128, 10.2 and 8.8, 238 of 4 behind 36 .. 357
// 26.6 and 24.6, 169 of 4 behind 100 .. 998 36.3 and 32.2; 183 of 2 behind 37 .. 375, 16 / 8 heads of 80, 26.8 and 28.5.
inline int order_keys(int64_t batch, int64_t pairs, int64_t table_keys, int head_dim, int64_t tile_wgs) {
  if (tile_wgs == 0 && pairs <= kUnits) return kNeverOrdered;
  const int64_t least = tile_wgs == 0 ? 140 : batch <= 64 ? 256 : batch <= 128 ? 440 : 1024;
  const int64_t by_pairs = tile_wgs == 0 || batch <= 64 ? pairs / 4 : batch <= 128 ? pairs * 3 / 4 : pairs * 4 / 3;
  const int64_t keys = (by_pairs > least ? by_pairs : least) * 128 / head_dim;
  if (table_keys <= keys) return kNeverOrdered;  // (a table this narrow says it without a look at the lengths,
  return batch <= 64 ? 0 : (int)keys;            // and the look costs what it saves where these fill one register)
}

#if defined(__HIP_DEVICE_COMPILE__)
// The largest value of a wave's lanes (none below 0), in all of them.
__device__ __forceinline__ int wave_max(int x) {
  auto with = [&](int other) { x = other > x ? other : x; };
  with(__builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  with(__builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  with(__builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  with(__builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  with(__builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  with(__builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// A workgroup's work: a share of a request's context for one KV head (f0 < 0), or a group of wave tiles of a request.
struct Work {
  int b, kv_head, q_start, q_len, kv_len, split, f0;
  int places, tail;  // of a chain, in wide workgroups: places that have work in all, and the first one from which on they are all chains
};

// This workgroup's work, found by every wave for itself from the lengths of the whole batch, which lie in REGS registers of its
// lanes; false for workgroups that have none.
// Batches without a context beyond order_keys keep the order of their requests: decode steps in the first batch * n_kv_heads *
// n_splits workgroups, which need only their own request's lengths, and the chains behind them.
// The order of the others.  A key tile takes a chunk's workgroup 1.1 us on a unit of its own, 1.5 beside another chain and 2.2 beside a
// decode step, which keeps the unit's memory path full.  So the chip is divided: on the first `units` compute units the
// workgroups of both layers (ids i and i + 256) are decode steps, the longest first in all, paired like those of
// attn_decode_kernel; on the others both are chains, the longest ones, a longer one with a shorter one.  What does not fit follows
// behind, shorter decode steps before shorter chains.
//   - The chains' part is as large as the groups of more than half of the longest chain need, since the kernel lasts as long as
//     its longest chain and these cannot start late; where decode steps fill more than a layer and are not much longer than the
//     chains (a decode step takes half as long per key, alone on its unit), at least what the decode steps leave of two layers.
//   - Decode steps of less than a layer whose contexts are shorter than the chunks' are done early: then the chains of the second
//     layer go beside them, and the longest have a unit for themselves (43 of 70 .. 708 tokens and 4 chunks of 192: 20.5 us, else 21.5).
//   - Without long chains the decode steps are what the kernel waits for, and all units start with them.
// Of split contexts only the shares that exist have a workgroup, so that chains start on the units that these leave free.
// us before (requests in batch order, empty shares among them; of the chains as many as the decode steps left slots for, beside each
// other) and now, 28 / 4 heads of 128: 96 decode steps of 180 .. 1800 tokens and 4 chunks of 512 63.8 -> 62, of 250 .. 2500 and 4 of
// 200 62.4 -> 50.8; 70 of 200 .. 2000 and 2 of 300 46.1 -> 33.7; 36 of 246 .. 2466 and 3 of 352 38.0 -> 31.9; 72 of 136 .. 1366 and 4 of
// 215 37.5 -> 28.6; 76 of 44 .. 441 and 4 of 72 15.6 -> 14.6; 20 of 240 .. 2408 and 4 of 68 21.1 -> 17.2; 5 of 97 .. 971 and 1 of 299
// 12.0 -> 11.1 (a scan over the requests through LDS took longer); 42 of 72 .. 723 and 4 of 64 12.4 -> 12.7 (decode steps whose lengths
// now come through the vector memory path; the largest loss of 96 mixes, their mean is 6 % faster).  Split contexts of very
// different lengths can lose more, since they are not ranked: 30 of 386 .. 3864 and one of 24 31.2 -> 33.7.
// A chain's chunk: up to kFewChunks chunks are ranked one by one, more by a search, whose time does not grow with their number.
// us, through the scan in LDS, one by one and by the search: 256 chunks of 32 tokens 130, 503 and 79; 100 decode steps and 100 chunks of
// 16 63, 139 and 55; 64 chunks of 100 53, 57 and 36; 16 of 512 215, 215 and 213; but a chunk of 64 alone 11.2, 10.4 and 10.8, 8 decode
// steps of 70 .. 709 and 2 chunks of 405 20.3, 19.6 and 19.9.
template <int REGS, bool WIDE>
__device__ __forceinline__ bool find_work(const PagedArgs& a, int id, Work& w) {
  const int lane = threadIdx.x & 63;
  const int table_keys = (int)((int64_t)a.max_blocks_per_seq << a.block_shift);
  const int pairs = a.batch * a.n_kv_heads;
  // this workgroup's place in the order of the batch
  auto in_batch_order = [&](int id) {
    w.split = a.n_splits > 1 ? id / pairs : 0;
    const int pair = id - w.split * pairs;
    w.b = pair / a.n_kv_heads;
    w.kv_head = pair - w.b * a.n_kv_heads;
    const const_table_t cu = (const_table_t)(uintptr_t)a.cu_seqlens_q, lens = (const_table_t)(uintptr_t)a.kv_lens;
    int start = cu[w.b], end = cu[w.b + 1], len = lens[w.b];
    asm volatile("" : "+s"(start), "+s"(end), "+s"(len));  // (asked for together)
    w.q_start = start;
    w.q_len = end - start;
    w.kv_len = len < table_keys ? len : table_keys;
    w.f0 = -1;
    return w.q_len > 0 && w.kv_len >= w.q_len && w.q_len * a.group <= kRows;
  };
  bool ordered = a.order_keys != kNeverOrdered;
  // WIDE: two of the first kind to a workgroup, number i from the front and from the back, one for each half of its waves
  const int half = WIDE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const int in_order = WIDE ? (pairs * a.n_splits + 1) / 2 : pairs * a.n_splits;
  auto unit_in_order = [&]() {
    if (!WIDE || half == 0) return in_batch_order(id);
    const int other = pairs * a.n_splits - 1 - id;
    return other > id && in_batch_order(other);
  };
  w.f0 = 0;
  if (!ordered && id < in_order) {
    w.f0 = -1;
    return unit_in_order();
  }

  int q_start[REGS], q_len[REGS], kv_len[REGS];
#pragma unroll
  for (int r = 0; r < REGS; ++r) kv_len[r] = a.kv_lens[r * 64 + lane < a.batch ? r * 64 + lane : a.batch - 1];
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    const int at = r * 64 + lane < a.batch ? r * 64 + lane : a.batch - 1;
    q_start[r] = a.cu_seqlens_q[at];
    q_len[r] = a.cu_seqlens_q[at + 1];
  }
  if (REGS > 1 && ordered) {
    bool far = false;  // (requests past the last one repeat it)
#pragma unroll
    for (int r = 0; r < REGS; ++r) far = far || kv_len[r] > a.order_keys;
    ordered = __builtin_amdgcn_ballot_w64(far) != 0;
    if (!ordered && id < in_order) {
      w.f0 = -1;
      return unit_in_order();
    }
  }

  int steps[REGS], groups[REGS];  // of a request of the first kind / of the second
  uint64_t chunks[REGS], any_chunk = 0, far_chunk = 0;
  int n_steps = 0, n_chunks = 0;
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    q_len[r] -= q_start[r];
    kv_len[r] = kv_len[r] < table_keys ? kv_len[r] : table_keys;
    if (r * 64 + lane >= a.batch || kv_len[r] < q_len[r]) q_len[r] = 0;  // (a context shorter than its new tokens is invalid)
    const bool many = q_len[r] * a.group > kRows, chunk = many && a.n_tile_wgs > 0;
    steps[r] = q_len[r] > 0 && !many ? (kv_len[r] + kDecodeKeys - 1) / kDecodeKeys : -1;
    groups[r] = chunk ? (((q_len[r] + kRows - 1) / kRows) * a.group + kWavesPerGroup - 1) / kWavesPerGroup : 0;
    n_steps += __builtin_popcountll(__builtin_amdgcn_ballot_w64(steps[r] > 0));
    chunks[r] = __builtin_amdgcn_ballot_w64(chunk);
    any_chunk |= chunks[r];
    n_chunks += __builtin_popcountll(chunks[r]);
    far_chunk |= __builtin_amdgcn_ballot_w64(chunk && kv_len[r] > kLongChain * kKvTileRows);
  }

  int step = -1, chain = -1, units = kFirstLayer, rows_wgs = 0, firsts = 0, shares[REGS];
  int chains = 0;  // (WIDE)
  if constexpr (WIDE) {
    int sum = 0;
#pragma unroll
    for (int r = 0; r < REGS; ++r) sum += groups[r];
    chains = __builtin_amdgcn_readlane(wave_scan_add(sum), 63) * a.n_kv_heads;
  }
  if (!ordered) {
    chain = id - in_order;
    w.places = in_order + chains;
    w.tail = in_order;
  } else {
    // workgroups of the first kind: one per share
    rows_wgs = n_steps * a.n_kv_heads;
    if (a.n_splits > 1) {
      int sum = 0;
#pragma unroll
      for (int r = 0; r < REGS; ++r) {
        int per;
        shares[r] = 0;
        if (steps[r] > 0) share_plan(steps[r], a.n_splits, a.least_log2, per, shares[r]);
        sum += shares[r];
      }
      rows_wgs = __builtin_amdgcn_readlane(wave_scan_add(sum), 63) * a.n_kv_heads;
    }
    if constexpr (WIDE) {
      int keys = 0;
#pragma unroll
      for (int r = 0; r < REGS; ++r) keys += steps[r] > 0 ? steps[r] : 0;
      const int all_steps = __builtin_amdgcn_readlane(wave_scan_add(keys), 63);
      // (numbers that shift the chains' places are multiples of 8: a KV head of a chunk keeps its dies)
      // one of the first kind to a workgroup as far as the chip has compute units, the longest ones, and two for the rest
      firsts = rows_wgs <= kUnits - chains ? rows_wgs : (rows_wgs + 1) / 2 > kUnits - chains ? (rows_wgs + 1) / 2 : kUnits - chains;
      const int n_rows = (firsts + 7) & ~7;
      int ahead = 0;
      if (rows_wgs > 0 && firsts + chains > kUnits) {
        // chains that last longer than a workgroup of the first kind go ahead of those, the others behind them
        const int tokens_of = (int)((float)all_steps * (float)a.n_kv_heads / (float)rows_wgs * kChainKeysPerStep);
        int far = 0;
#pragma unroll
        for (int r = 0; r < REGS; ++r) {
          int tokens = kv_len[r] - tokens_of;
          tokens = tokens < 0 ? 0 : tokens < q_len[r] ? tokens : q_len[r];
          far += groups[r] > 0 ? (int)((float)groups[r] * tokens / q_len[r]) : 0;
        }
        ahead = __builtin_amdgcn_readlane(wave_scan_add(far), 63) * a.n_kv_heads & ~7;
        const int most = ((int)gridDim.x - n_rows - kTrailing) & ~7;  // (the grid has room for these)
        ahead = ahead < most ? ahead : most;
      }
      w.places = n_rows + chains;
      w.tail = ahead + n_rows;
      if (id < ahead) {
        chain = id;
      } else if (id < ahead + n_rows) {
        step = id - ahead;
        if (step >= firsts) step = rows_wgs;  // (a place that only rounds the number up)
        else if (half == 1) step = 2 * firsts - 1 - step;
      } else {
        chain = id - n_rows;
      }
    } else {
      // (a multiple of 8, like everything that shifts the chains' places: a KV head of a chunk keeps its dies)
      bool beside_steps = false;
      if (rows_wgs == 0) {
        beside_steps = true;  // (chains only)
      } else if (far_chunk != 0 || (any_chunk != 0 && id >= kFirstLayer)) {
        int longest = 0;
        uint64_t longer = 0, far_longer = 0;
#pragma unroll
        for (int r = 0; r < REGS; ++r) longest = groups[r] > 0 && kv_len[r] > longest ? kv_len[r] : longest;
        longest = wave_max(longest);
#pragma unroll
        for (int r = 0; r < REGS; ++r) longer |= __builtin_amdgcn_ballot_w64(steps[r] > 0 && kv_len[r] > longest);
        beside_steps = rows_wgs <= kFirstLayer && longer == 0;
        if (far_chunk != 0 && !beside_steps) {
          int far = 0;  // groups whose chains are longer than half of the longest
#pragma unroll
          for (int r = 0; r < REGS; ++r) {
            int tokens = kv_len[r] - longest / 2;
            tokens = tokens < 0 ? 0 : tokens < q_len[r] ? tokens : q_len[r];
            far += groups[r] > 0 ? (int)((float)groups[r] * tokens / q_len[r]) : 0;
            far_longer |= __builtin_amdgcn_ballot_w64(steps[r] > 0 && kv_len[r] - longest / 2 > longest);
          }
          int chain_units = __builtin_amdgcn_readlane(wave_scan_add(far), 63) * a.n_kv_heads / 2;
          if (far_longer == 0 && rows_wgs > kFirstLayer && chain_units < (2 * kFirstLayer - rows_wgs) / 2) chain_units = (2 * kFirstLayer - rows_wgs) / 2;
          chain_units = (chain_units < kFirstLayer - kStepUnits ? chain_units : kFirstLayer - kStepUnits) & ~7;
          units = kFirstLayer - chain_units;
        }
      }
      if (any_chunk != 0 && units > rows_wgs) units = (rows_wgs + 7) & ~7;
      const int chain_units = kFirstLayer - units;

      if (id < units) {
        step = id;
      } else if (id < kFirstLayer || beside_steps) {
        chain = id - units;
      } else if (id < kFirstLayer + units) {
        step = units + id - kFirstLayer;
        if (step >= rows_wgs) chain = 2 * chain_units + step - (rows_wgs > units ? rows_wgs : units);
      } else if (id < 2 * kFirstLayer) {
        const int at = id - (kFirstLayer + units);  // (the longer the first chain of a unit, the shorter the second)
        chain = 2 * chain_units - 8 - (at & ~7) + (at & 7);
      } else {
        step = 2 * units + id - 2 * kFirstLayer;
        if (step >= rows_wgs) chain = id - (rows_wgs > units ? rows_wgs : units);
      }
    }
  }

  if (chain >= 0) {
    const int target = chain / a.n_kv_heads;
    w.kv_head = chain - target * a.n_kv_heads;
    w.split = 0;
    w.b = -1;
    auto take = [&](int r, int j, int groups_left) {  // lane j of register r, from the last group down
      w.b = r * 64 + j;
      w.q_start = __builtin_amdgcn_readlane(q_start[r], j);
      w.q_len = __builtin_amdgcn_readlane(q_len[r], j);
      w.kv_len = __builtin_amdgcn_readlane(kv_len[r], j);
      w.f0 = (groups_left - 1) * kWavesPerGroup;
    };
    if (n_chunks <= kFewChunks) {
      int before[REGS];  // groups ahead of this lane's chunk: those of chunks with longer contexts
#pragma unroll
      for (int r = 0; r < REGS; ++r) before[r] = 0;
#pragma unroll
      for (int r = 0; r < REGS; ++r)
        for (uint64_t left = chunks[r]; left != 0; left &= left - 1) {
          const int j = __builtin_ctzll(left);
          const int kv = __builtin_amdgcn_readlane(kv_len[r], j), n = __builtin_amdgcn_readlane(groups[r], j);
#pragma unroll
          for (int e = 0; e < REGS; ++e) before[e] += kv > kv_len[e] || (kv == kv_len[e] && r * 64 + j < e * 64 + lane) ? n : 0;
        }
#pragma unroll
      for (int r = 0; r < REGS; ++r) {
        const uint64_t here = __builtin_amdgcn_ballot_w64(groups[r] > 0 && before[r] <= target && target < before[r] + groups[r]);
        if (here != 0) {
          const int j = __builtin_ctzll(here);
          take(r, j, __builtin_amdgcn_readlane(before[r] + groups[r], j) - target);
        }
      }
      return w.b >= 0;  // (past the last group otherwise)
    }
    // More chunks are taken by their key tiles, most first and equal ones by number: a search over the bits of a number of tiles,
    // which adds up the groups of all chunks that reach it.
    int tiles[REGS], most = 0, all = 0, v = 0, ahead = 0;  // ahead: groups of the chunks with more than v tiles
#pragma unroll
    for (int r = 0; r < REGS; ++r) {
      tiles[r] = groups[r] > 0 ? (kv_len[r] + kKvTileRows - 1) / kKvTileRows : 0;
      most = tiles[r] > most ? tiles[r] : most;
      all += groups[r];
    }
    if (target >= __builtin_amdgcn_readlane(wave_scan_add(all), 63)) return false;  // past the last group
    most = wave_max(most);  // (at least 1: there are chunks)
    for (int bit = 1 << (31 - __builtin_clz(most)); bit > 0; bit >>= 1) {
      int sum = 0;
#pragma unroll
      for (int r = 0; r < REGS; ++r) sum += tiles[r] >= (v | bit) ? groups[r] : 0;
      sum = __builtin_amdgcn_readlane(wave_scan_add(sum), 63);
      if (sum > target) v |= bit;
      else ahead = sum;
    }
    int at = target - ahead;  // among the groups of the chunks with v tiles
#pragma unroll
    for (int r = 0; r < REGS; ++r) {
      const int mine = v > 0 && tiles[r] == v ? groups[r] : 0;
      const int upto = wave_scan_add(mine);
      const uint64_t here = __builtin_amdgcn_ballot_w64(upto - mine <= at && at < upto);
      if (w.b < 0 && here != 0) {
        const int j = __builtin_ctzll(here);
        take(r, j, __builtin_amdgcn_readlane(upto, j) - at);
      }
      at -= __builtin_amdgcn_readlane(upto, 63);
    }
    return w.b >= 0;
  }

  w.f0 = -1;
  if (step >= rows_wgs) return false;
  w.split = 0;
  // ranked by context, or (where all of them start together, and where contexts are split: ranked, the second workgroups of the
  // units with the longest shares had long ones too, 20 decode steps of 240 .. 2408 tokens and 4 chunks of 68 21.2 -> 23.3 us)
  // just the request number `rank` of this kind
  const bool ranked = rows_wgs > (WIDE ? firsts : units) && a.n_splits == 1;
  uint64_t of_kind[REGS];
#pragma unroll
  for (int r = 0; r < REGS; ++r) of_kind[r] = __builtin_amdgcn_ballot_w64(steps[r] > 0);
  int pair = !WIDE && ranked && step < units ? units - 1 - step : step;  // (see attn_decode_kernel)
  if (a.n_splits > 1) {
    // share-major: the first shares of all pairs, then the second shares of those that have one, ...
    for (;;) {
      int n = 0;
#pragma unroll
      for (int r = 0; r < REGS; ++r) n += __builtin_popcountll(of_kind[r]);
      n *= a.n_kv_heads;
      if (pair < n || n == 0) break;
      pair -= n;
      ++w.split;
#pragma unroll
      for (int r = 0; r < REGS; ++r) of_kind[r] = __builtin_amdgcn_ballot_w64(shares[r] > w.split);
    }
  }
  const int rank = pair / a.n_kv_heads;
  w.kv_head = pair - rank * a.n_kv_heads;
  w.b = ranked ? search_rank(steps, rank, table_keys) : -1;
  int skip = rank;
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    if (!ranked) {
      const int n = __builtin_popcountll(of_kind[r]);
      if (skip >= 0 && skip < n) w.b = r * 64 + nth_lane(of_kind[r], skip);
      skip -= n;
    }
    if (w.b / 64 == r) {
      w.q_start = __builtin_amdgcn_readlane(q_start[r], w.b % 64);
      w.q_len = __builtin_amdgcn_readlane(q_len[r], w.b % 64);
      w.kv_len = __builtin_amdgcn_readlane(kv_len[r], w.b % 64);
    }
  }
  return true;
}

#endif  // __HIP_DEVICE_COMPILE__

// LDS of a workgroup: the stages of the plain and the packed-rows form (of a wide one's halves, each its own), or the pipeline's rings.
template <int D, bool WIDE>
struct PagedLds {
  static constexpr int kHalf = (StageGeom<D>::kLdsBytes + 1023) / 1024 * 1024;
  static constexpr int kRows = (WIDE ? kHalf : 0) + StageGeom<D>::kLdsBytes, kRings = TileGeom<D, 1, WIDE ? kWavesPerItem * kWaveTileRows : 0>::kLdsBytes;
  static constexpr int kBytes = kRows > kRings ? kRows : kRings;
};

#if defined(__HIP_DEVICE_COMPILE__)
// A group of four wave tiles of a request (f0 .. f0 + 3 for one KV head) in the plain form: the first four waves of the workgroup.
template <int D>
__device__ __forceinline__ void run_plain(const PagedArgs& a, unsigned char* smem, int b, int kv_head, int q_start, int q_len, int kv_len, int f0) {
  using G = StageGeom<D>;
  const int32_t* table = a.block_tables + (int64_t)b * a.max_blocks_per_seq;
  const int n_wave_tiles = (q_len + kRows - 1) / kRows * a.group;
  const int shift = kv_len - q_len;  // keys that precede the first new token
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = lane & 31;

  // this wave's tile
  const bool works = wave < kWavesPerGroup;  // (not the loading waves of a wide workgroup)
  int f = f0 + wave;
  const bool active = works && f < n_wave_tiles;
  if (!active) f = n_wave_tiles - 1;
  const int tok_tile = f / a.group;
  const int head = kv_head * a.group + (f - tok_tile * a.group);
  const int q0 = tok_tile * kRows;
  const int f_last = (f0 + kWavesPerGroup - 1 < n_wave_tiles ? f0 + kWavesPerGroup - 1 : n_wave_tiles - 1);
  // keys visible to the last new token of a tile that starts at q: shift + min(q + 32, q_len)
  auto keys_of_tile = [&](int q) { return shift + (q + kRows < q_len ? q + kRows : q_len); };
  const int tiles_wg = (keys_of_tile((f_last / a.group) * kRows) + kKvTileRows - 1) / kKvTileRows;
  const int tiles_wave = active ? (keys_of_tile(q0) + kKvTileRows - 1) / kKvTileRows : 0;

  // first K/V tile in flight before anything else, and the second tile's block-table lookup behind it
  TileSlots<D, kKvTileRows, kWavesPerGroup> slots, next_slots;
  if (works) {
    fetch_tile_slots(slots, a, table, wave, lane, kv_len, 0);
    issue_tile_loads(slots, a, smem, wave, lane, kv_head);
  }
  if (works && 1 < tiles_wg) fetch_tile_slots(slots, a, table, wave, lane, kv_len, kKvTileRows);

  WaveTile<D, 1> w;
  w.init(lane, a.scale_log2);
  int row = q0 + m;
  row = row < q_len ? row : q_len - 1;
  w.load_q(0, a.q + (int64_t)(q_start + row) * a.q_stride + head * D, shift + row);
  const int min_lim = shift + q0;  // smallest limit among the tile's tokens

  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  for (int t = 0; t < tiles_wg; ++t) {
    unsigned char* stage = smem + (t & 1) * G::kStageBytes;
    // tile t + 1 is fetched (its slots arrived during the previous iteration) and tile t + 2 is looked up
    // while tile t is used
    if (works && t + 1 < tiles_wg) issue_tile_loads(slots, a, smem + ((t + 1) & 1) * G::kStageBytes, wave, lane, kv_head);
    if (works && t + 2 < tiles_wg) fetch_tile_slots(next_slots, a, table, wave, lane, kv_len, (t + 2) * kKvTileRows);
    if (t < tiles_wave) {
      const int kv0 = t * kKvTileRows;
      w.template tile<2>(stage, kv0, kv0 + kKvTileRows - 1 > min_lim);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    slots = next_slots;
  }
  w.store_row(0, active && q0 + m < q_len ? a.out + ((int64_t)(q_start + q0 + m) * a.n_q_heads + head) * D : nullptr);
}

// A workgroup, from its place in the grid to its result.
template <int D, bool WIDE>
__device__ __forceinline__ void run_place(const PagedArgs& a, unsigned char* smem, float* s_stats) {
  const int tid = (int)threadIdx.x;
  using G = StageGeom<D>;
  using Source = PagedSource<WIDE ? 4 : 0>;
  constexpr int kHalfLds = PagedLds<D, WIDE>::kHalf;
  // new tokens and context of request b (context cut to what the table can describe; q_len 0: nothing to do,
  // also for a context shorter than its new tokens, which is invalid)
  auto lengths_of = [&](int b, int& q_len, int& kv_len) {
    q_len = a.cu_seqlens_q[b + 1] - a.cu_seqlens_q[b];
    kv_len = a.kv_lens[b];
    const int64_t table_keys = (int64_t)a.max_blocks_per_seq << a.block_shift;
    if (kv_len > table_keys) kv_len = (int)table_keys;
    if (q_len < 0 || kv_len < q_len) q_len = 0;
  };
  int b, kv_head, q_start, q_len, kv_len, split = 0, f0 = -1;  // f0 < 0: the packed-rows form or the decode form
  int places = 0, tail = 0;
  if (WIDE || a.batch <= kOrderedMost) {
    Work w;
    bool found;
    if constexpr (WIDE) {
      found = a.batch <= 64 ? find_work<1, true>(a, (int)blockIdx.x, w) : find_work<2, true>(a, (int)blockIdx.x, w);
    } else {
      found = a.batch <= 64 ? find_work<1, false>(a, (int)blockIdx.x, w) : a.batch <= 128 ? find_work<2, false>(a, (int)blockIdx.x, w) : find_work<4, false>(a, (int)blockIdx.x, w);
    }
    if (!found) {
      if (WIDE && w.f0 < 0) __syncthreads();  // (the other half of the waves may have a decode step)
      return;
    }
    b = w.b, kv_head = w.kv_head, q_start = w.q_start, q_len = w.q_len, kv_len = w.kv_len, split = w.split, f0 = w.f0, places = w.places, tail = w.tail;
  } else {
    const int n_rows_wgs = (int)gridDim.x - a.n_tile_wgs;
    // This workgroup's place: decode steps, then chains.  Where the decode steps fill the first layer of the chip (256 units) and
    // part of the second, the second layer's remaining slots go to the longest chunk chains, and a chain that shares its
    // unit with a decode step crawls: the decode step keeps the unit's memory path full (a key tile takes the chain 2.2 us
    // instead of 1.5).  When the batch has long chains, those slots are moved: c chains end the first layer and c lie
    // above them in the second, so that chains share units with chains and decode steps with decode steps (96 decode
    // steps and 4 chunks of 512 with up to 3 chunks behind them: 71.3 -> 62 us; over 48 mixes +5 %, from +17 to -3).
    // Without long chains the decode steps are what the kernel waits for, and they stay in front.
    int place = (int)blockIdx.x;
    {
      int c = (kFirstLayer * 2 - n_rows_wgs) / 2;
      c = (c < a.n_tile_wgs ? c : a.n_tile_wgs) & ~7;  // (places only change hands with ids that the grid has; a multiple of 8: KV heads keep their dies)
      if (n_rows_wgs > kFirstLayer && n_rows_wgs < 2 * kFirstLayer && place >= kFirstLayer - c && place < n_rows_wgs + c) {
        bool far = false;
        for (int r = (int)threadIdx.x; r < a.batch; r += 256) {
          int q_len, kv_len;
          lengths_of(r, q_len, kv_len);
          far = far || (q_len * a.group > kRows && kv_len > kLongChain * kKvTileRows);
        }
        if (__syncthreads_or(far)) place = place < kFirstLayer ? n_rows_wgs + place - (kFirstLayer - c) : place - c;
      }
    }
    if (place < n_rows_wgs) {
      const int r = place;
      // (share-major: the workgroups of the first shares, which every request has, lie next to each other and are dealt
      // to all dies alike; the further shares, some of them empty when contexts differ in length, come behind them)
      const int pairs = a.batch * a.n_kv_heads;
      split = r / pairs;
      const int pair = r - split * pairs;
      b = pair / a.n_kv_heads;
      kv_head = pair - b * a.n_kv_heads;
      lengths_of(b, q_len, kv_len);
      if (q_len == 0 || q_len * a.group > kRows) return;
    } else{
      // which group of which request: see above.  Thread i adds up requests [i * per, (i + 1) * per).
      int* s_scan = reinterpret_cast<int*>(s_stats);  // [0..3] the waves' groups, [4..7] the waves' requests, [256] = request, [257] = group
      const int target = (place - n_rows_wgs) / a.n_kv_heads;
      kv_head = (place - n_rows_wgs) - target * a.n_kv_heads;
      const int per = (a.batch + 255) / 256;
      auto groups_of = [&](int r, int& kv_len) {
        int q_len;
        lengths_of(r, q_len, kv_len);
        if (q_len * a.group <= kRows) return 0;
        return (((q_len + kRows - 1) / kRows) * a.group + kWavesPerGroup - 1) / kWavesPerGroup;
      };
      const int first = (int)threadIdx.x * per, last = first + per < a.batch ? first + per : a.batch;
      int mine = 0, mine_reqs = 0;  // groups, and requests that have groups, in this thread's slice
      for (int r = first; r < last; ++r) {
        int kv;
        const int n = groups_of(r, kv);
        mine += n;
        mine_reqs += n > 0 ? 1 : 0;
      }
      const int lane_ = threadIdx.x & 63, wave_ = threadIdx.x >> 6;
      int incl = mine, incl_reqs = mine_reqs;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d), up_reqs = __shfl_up(incl_reqs, d);
        if (lane_ >= d) {
          incl += up;
          incl_reqs += up_reqs;
        }
      }
      if (lane_ == 63) {
        s_scan[wave_] = incl;
        s_scan[4 + wave_] = incl_reqs;
      }
      if (threadIdx.x == 0) s_scan[256] = -1;
      __syncthreads();
      int before = incl - mine, before_reqs = incl_reqs - mine_reqs;  // of the slices ahead of this thread's
      for (int i = 0; i < wave_; ++i) {
        before += s_scan[i];
        before_reqs += s_scan[4 + i];
      }
      const int total_reqs = s_scan[4] + s_scan[5] + s_scan[6] + s_scan[7];
      if (target >= s_scan[0] + s_scan[1] + s_scan[2] + s_scan[3]) return;  // past the last group
      // Requests with the longest contexts first: their workgroups run longest, and the kernel is as long as the
      // last of them.  The requests of this form (few: prefill chunks) are gathered in LDS, ranked by context
      // length, and the groups are counted off in that order.  (More than kMaxSorted of them: batch order.)
      constexpr int kMaxSorted = 256;
      if (total_reqs <= kMaxSorted) {
        int* s_req = reinterpret_cast<int*>(smem);  // the tile stages are not in use yet
        int* s_groups = s_req + kMaxSorted, *s_key = s_req + 2 * kMaxSorted;
        int* s_sorted_req = s_req + 3 * kMaxSorted, *s_sorted_groups = s_req + 4 * kMaxSorted;
        int k = before_reqs;
        for (int r = first; r < last; ++r) {
          int kv;
          const int n = groups_of(r, kv);
          if (n > 0) {
            s_req[k] = r;
            s_groups[k] = n;
            s_key[k] = kv;
            ++k;
          }
        }
        __syncthreads();
        if ((int)threadIdx.x < total_reqs) {
          const int key = s_key[threadIdx.x];
          int rank = 0;
          for (int j = 0; j < total_reqs; ++j) rank += (s_key[j] > key || (s_key[j] == key && j < (int)threadIdx.x)) ? 1 : 0;
          s_sorted_req[rank] = s_req[threadIdx.x];
          s_sorted_groups[rank] = s_groups[threadIdx.x];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
          int at = 0;
          for (int e = 0; e < total_reqs; ++e) {
            const int n = s_sorted_groups[e];
            if (target < at + n) {
              s_scan[256] = s_sorted_req[e];
              s_scan[257] = n - 1 - (target - at);  // from the last group down
              break;
            }
            at += n;
          }
        }
      } else if (target >= before && target < before + mine) {
        int at = before;
        for (int r = first; r < last; ++r) {
          int kv;
          const int n = groups_of(r, kv);
          if (target < at + n) {
            s_scan[256] = r;
            s_scan[257] = n - 1 - (target - at);
            break;
          }
          at += n;
        }
      }
      __syncthreads();
      b = __builtin_amdgcn_readfirstlane(s_scan[256]);
      if (b < 0) return;  // (cannot happen: the target was below the total)
      f0 = __builtin_amdgcn_readfirstlane(s_scan[257]) * kWavesPerGroup;
      __syncthreads();  // (the scan area is the packed-rows form's statistics area, the lists lie in the tile stages)
    }
    if (place >= n_rows_wgs) lengths_of(b, q_len, kv_len);
    q_start = a.cu_seqlens_q[b];
  }
  if (f0 < 0) {
    const int half = WIDE ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0, thread = tid - 256 * half;
    unsigned char* const lds = smem + half * kHalfLds;
    bool met;  // (the halves of a wide workgroup share one barrier)
    if constexpr (kDecodeForm<D>) {
      if (q_len * a.group <= kDecodeRows && (1 << a.block_shift) >= kDecodeMinBlock) {
        met = run_decode<D>(a, reinterpret_cast<float*>(lds), kWavesPerGroup, kWavesPerGroup, b, kv_head, q_start, q_len, kv_len, split, thread);
        if (WIDE && !met) __syncthreads();
        return;
      }
    }
    met = run_packed_rows<D>(a, lds, s_stats + half * (2 * kWavesPerGroup * 64), a.block_tables + (int64_t)b * a.max_blocks_per_seq, q_start, q_len, kv_len, kv_head, b, split,
                             thread);
    if (WIDE && !met) __syncthreads();
    return;
  }
  const int32_t* table = a.block_tables + (int64_t)b * a.max_blocks_per_seq;
  if (f0 >= (q_len + kRows - 1) / kRows * a.group) return;  // (cannot happen: the group was counted from these lengths)
  bool redo = true;

  // The group runs on the packed kernel's pipeline when the cache layout allows (see PagedSource); if its row sums
  // leave that path's range, or the layout does not allow, the plain loop below computes (or recomputes) it.
  if constexpr (TileLoader<D>::kUniformStep) {
    if ((1 << a.block_shift) >= PagedSource<0>::Gather<D>::kRowsPerInstr && a.num_blocks <= (0x7fffffff >> a.block_shift)) {
      Source src;
      src.args = &a;
      src.table = table;
      src.q_start = q_start;
      src.q_len = q_len;
      src.kv_len = kv_len;
      src.f0 = f0;
      src.kv_head = kv_head;
      AttnArgs fa;
      fa.q = a.q;
      fa.k = nullptr;
      fa.v = nullptr;
      fa.out = a.out;
      fa.q_stride = a.q_stride;
      fa.k_stride = 0;
      fa.v_stride = 0;
      fa.cu_seqlens = nullptr;
      fa.items = nullptr;
      fa.ctrl = nullptr;
      fa.n_q_heads = a.n_q_heads;
      fa.group = a.group;
      fa.scale_log2 = a.scale_log2;
      int* s_claim = reinterpret_cast<int*>(s_stats);  // (unused by a paged item; the redo flag lives behind it)
      if (!attn_item_loop<D, true>(fa, src, smem, s_claim, s_claim + 8)) {
        if (!WIDE || places <= (int)gridDim.x) return;
        redo = false;
      }
    }
  }
  if (redo) run_plain<D>(a, smem, b, kv_head, q_start, q_len, kv_len, f0);
  if constexpr (WIDE) {
    // The host sizes a wide grid for the places that it takes the batch to have (wide_grid).  One that has more, because its chunks are
    // not the whole ones that their tokens look like or because some requests have no new token, leaves the places past the grid's
    // end to the last workgroups, all of them chains, through the plain loop, whose code is here anyway (and which gives other last bits).
    const int last = (int)gridDim.x - 1 - (int)blockIdx.x, workers = (int)gridDim.x - tail;
    for (int id = (int)gridDim.x + last; last < workers && id < places; id += workers) {
      Work w;
      if (!(a.batch <= 64 ? find_work<1, true>(a, id, w) : find_work<2, true>(a, id, w)) || w.f0 < 0) return;  // (cannot happen: a chain's place)
      __syncthreads();
      run_plain<D>(a, smem, w.b, w.kv_head, w.q_start, w.q_len, w.kv_len, w.f0);
    }
  }
}

#endif

template <int D, bool WIDE>
__global__ __launch_bounds__(WIDE ? 512 : 256) __attribute__((amdgpu_waves_per_eu(kPagedWavesPerSimd, kPagedWavesPerSimd))) void attn_paged_kernel(const PagedArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[PagedLds<D, WIDE>::kBytes];
  __shared__ float s_stats[(WIDE ? 2 : 1) * 2 * kWavesPerGroup * 64];
  if constexpr (kDecodeForm<D>) static_assert(kWavesPerGroup * kDecodeLdsPerWave<D> <= (size_t)StageGeom<D>::kLdsBytes, "the decode form fits the tile stages");
  ask_for_arguments(a);
  asm volatile("" : : "s"(a.n_tile_wgs), "s"(a.order_keys));
  run_place<D, WIDE>(a, smem, s_stats);
#else
  (void)a;
#endif
}

// Merges the partial results of split contexts (n_splits > 1).  grid = (n_kv_heads, batch, parts), kCombineThreads<GROUPS> threads;
// parts: as many as give every thread 4 output columns of one row, for the most rows a request of the batch can have.
// Requests that took the wave-tile form, have no new tokens, or whose context fits one share (already finished by one
// workgroup) are skipped.
// The kernel runs on an idle chip, and latency is all it costs, most of it the launch, the lengths and the fetch of its own code.  So it
// asks for everything it needs (every share's row statistics and columns) before it uses any of it, one round trip to memory behind the
// lengths; and it has little code on any way through: GROUPS threads have the same columns, each with every GROUPS-th share, up to EACH
// of them, in code for 2, 4 or EACH, and the first adds up what they have through LDS.  us of both kernels, with one thread for all of up
// to 16 shares and so (before ask_for_arguments and `quotient`), 28 / 4 heads of 128: 4 requests of 300 .. 1500 tokens 7.7 -> 6.9, 8 of 750 .. 1500 9.3 -> 8.6, 32 of 750 .. 1500
// (2 shares) 18.8 -> 17.6, 4 of 8000 .. 16000 22.3 -> 21.5; two shares for each of eight waves instead of four for each of four 7.1 where
// four have 6.9, four for each of sixteen 9.5 where eight for each of eight have 8.5, which take 8.2 with the shorter ways beside the long one.
// With one workgroup per (request, KV head) a request of more than 8 rows of 128 took that trip two to four times: 30 requests of 4 new
// tokens, 28 / 4 heads of 128, 29.1 -> 27.2 us; 20 of 2, 28 / 2 heads, 18.9 -> 15.9.
// The records of all shares asked for together with the lengths, whether they exist or not, cost what they gave: one request of 6000
// tokens 10.9 -> 10.5 us of both kernels, 4 of 50 .. 300 under a table of 8192 keys 7.3 -> 7.1, but of contexts that are not cut 40 of
// 100 .. 500 under such a table 9.3 -> 10.1, 16 of 50 .. 400 7.9 -> 8.4 (out of the caches 12.1 -> 13.6).
// Shares of a context.  16 left a lone request with a quarter of the chip: 28 / 4 heads of 128, one of 16 384 tokens 18.5 -> 11.3 us (10.7 now), of
// 5000 10.2 -> 8.2 (7.6), two of 16 000 19.0 -> 15.5 (14.9); beside chunks there are 16 still (choose_splits).
constexpr int kMaxSplits = 64;
template <int GROUPS>
constexpr int kCombineThreads = GROUPS > 4 ? 64 * GROUPS : 256;
template <int GROUPS>
constexpr int kCombinePieces = kCombineThreads<GROUPS> / GROUPS;  // of 4 columns of a row that a workgroup does

#if defined(__HIP_DEVICE_COMPILE__)
template <int D, int GROUPS, int EACH>
__device__ __forceinline__ void merge_shares(const PagedArgs& a, const float* recs, int n_shares, int q_start, int kv_head, int n_rows, int parts) {
  constexpr int kColGroups = D / 4, kPieces = kCombinePieces<GROUPS>;
  static_assert(kPieces % 64 == 0, "whole waves");
  const int group = GROUPS == 1 ? 0 : (int)threadIdx.x / kPieces, piece = (int)threadIdx.x % kPieces;
  const int pieces = n_rows * kColGroups;
  for (int base = (int)blockIdx.z * kPieces; base < pieces; base += parts * kPieces) {
    const int i = base + piece;
    if (GROUPS == 1 && i >= pieces) return;
    const int row = i < pieces ? i / kColGroups : 0, col = (i % kColGroups) * 4;
    f32x4_t v[EACH];
    float top[EACH], sum[EACH];
    // (shares past the last one re-read it and are left out below: no branch between the loads)
#pragma unroll
    for (int s = 0; s < EACH; ++s) {
      const int share = s * GROUPS + group;
      const float* rec = recs + (int64_t)(share < n_shares ? share : n_shares - 1) * kPartialFloats<D>;
      top[s] = rec[row];
      sum[s] = rec[kRows + row];
      v[s] = *reinterpret_cast<const f32x4_t*>(rec + 2 * kRows + row * D + col);
    }
    float best = top[0];
#pragma unroll
    for (int s = 1; s < EACH; ++s) best = fmaxf(best, top[s]);
    float total = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < EACH; ++s) {
      // (not by weight 0 alone: an infinite V in the last share would come out as NaN)
      const bool live = s * GROUPS + group < n_shares;
      const float w = live ? fast_exp2((top[s] - best) * a.scale_log2) : 0.f;
      total += w * (live ? sum[s] : 0.f);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += w * (live ? v[s][e] : 0.f);
    }
    if constexpr (GROUPS > 1) {
      __shared__ f32x4_t s_acc[GROUPS][kPieces];
      __shared__ f32x2_t s_stat[GROUPS][kPieces];
      s_acc[group][piece] = acc;
      s_stat[group][piece] = f32x2_t{best, total};
      __syncthreads();
      if (group == 0) {
        f32x2_t stat[GROUPS];
        f32x4_t part[GROUPS];
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
          stat[g] = s_stat[g][piece];
          part[g] = s_acc[g][piece];
        }
#pragma unroll
        for (int g = 1; g < GROUPS; ++g) best = fmaxf(best, stat[g][0]);
        total = 0.f;
        acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
          const float w = g < n_shares ? fast_exp2((stat[g][0] - best) * a.scale_log2) : 0.f;
          total += w * stat[g][1];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] += w * part[g][e];
        }
      }
      __syncthreads();  // (before the next pieces' results)
      if (group != 0 || i >= pieces) continue;
    }
    const float inv = 1.0f / total;
    const int token = quotient(row, a.group);
    const int head = kv_head * a.group + (row - token * a.group);
    const f32x2_t a0 = {acc[0] * inv, acc[1] * inv}, a1 = {acc[2] * inv, acc[3] * inv};
    u32x2_t pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector(a0, bf16x2_t)),
                  __builtin_bit_cast(uint32_t, __builtin_convertvector(a1, bf16x2_t))};
    *reinterpret_cast<u32x2_t*>(a.out + ((int64_t)(q_start + token) * a.n_q_heads + head) * D + col) = pk;
  }
}
#endif

template <int D, int GROUPS, int EACH>
__global__ __launch_bounds__(kCombineThreads<GROUPS>) void attn_paged_combine_kernel(const PagedArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  const int b = blockIdx.y, kv_head = blockIdx.x;
  const const_table_t cu = (const_table_t)(uintptr_t)a.cu_seqlens_q, lens = (const_table_t)(uintptr_t)a.kv_lens;
  int parts = (int)gridDim.z;
  asm volatile("" : "+s"(parts));
  ask_for_arguments(a);
  int q_start = cu[b], q_end = cu[b + 1], kv_len = lens[b];
  asm volatile("" : "+s"(q_start), "+s"(q_end), "+s"(kv_len));  // (asked for together)
  const int q_len = q_end - q_start;
  const int64_t table_keys = (int64_t)a.max_blocks_per_seq << a.block_shift;
  if (kv_len > table_keys) kv_len = (int)table_keys;
  if (q_len <= 0 || kv_len < q_len || q_len * a.group > kRows) return;
  const int n_rows = q_len * a.group;
  const int n_halves = (kv_len + kKvTileRows / 2 - 1) / (kKvTileRows / 2);
  int per_share, n_shares;
  share_plan(n_halves, a.n_splits, a.least_log2, per_share, n_shares);
  if (n_shares == 1) return;  // done by one workgroup, which wrote the output itself
  const float* recs = a.partials + ((int64_t)b * a.n_kv_heads + kv_head) * a.n_splits * kPartialFloats<D>;
  if (EACH > 2 && n_shares <= 2 * GROUPS) merge_shares<D, GROUPS, 2>(a, recs, n_shares, q_start, kv_head, n_rows, parts);
  else if (EACH > 4 && n_shares <= 4 * GROUPS) merge_shares<D, GROUPS, 4>(a, recs, n_shares, q_start, kv_head, n_rows, parts);
  else merge_shares<D, GROUPS, EACH>(a, recs, n_shares, q_start, kv_head, n_rows, parts);
#else
  (void)a;
#endif
}

}  // namespace paged
}  // namespace hydra
