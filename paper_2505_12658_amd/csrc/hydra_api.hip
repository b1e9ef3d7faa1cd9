// C ABI of the library: argument validation on the host, then launches.  See include/hydra_attn.h
// for the contract of every entry point.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <tuple>
#include <type_traits>

#include "../../include/hydra_attn.h"
#include "attn_fwd.hpp"
#include "attn_paged.hpp"
#include "batch_rules.hpp"
#include "kv_write.hpp"
#include "page_cache.hpp"
#include "worklist.hpp"

static_assert(hydra::rules::kTileTokens == hydra::kWaveTileRows && hydra::rules::kTileKeys == hydra::kKvTileRows && hydra::rules::kTileTokens == hydra::paged::kRows &&
                  hydra::rules::kChainTiles == hydra::paged::kWavesPerGroup && hydra::rules::kUnits == hydra::paged::kUnits && hydra::rules::kTrailing == hydra::paged::kTrailing,
              "what the kernels have");

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool head_dim_supported(int d) { return d == 64 || d == 80 || d == 128; }

// Enqueues one kernel and returns the status of THIS launch (the runtime's sticky last-error slot
// is shared by every caller of the process and may hold somebody else's failure).
template <typename... Params, typename... Args>
hipError_t launch_lds(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds_bytes, hipStream_t stream, const Args&... args) {
  static_assert(sizeof...(Params) == sizeof...(Args), "one argument per kernel parameter");
  std::tuple<Params...> vals(args...);
  return std::apply(
      [&](auto&... v) {
        void* ptrs[] = {static_cast<void*>(&v)...};
        return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, ptrs, lds_bytes, stream);
      },
      vals);
}
template <typename... Params, typename... Args>
hipError_t launch(void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t stream, const Args&... args) {
  return launch_lds(kernel, grid, block, 0, stream, args...);
}

// A row-copy kernel (its form for rows of whole kilobytes, its form for others) over `rows` rows of row16 pieces: one launch,
// or several where a grid cannot hold them.
template <typename Args>
hipError_t launch_row_copy(void (*kilobytes)(Args), void (*others)(Args), Args args, int32_t rows, int32_t row16, hipStream_t stream) {
  args.rows = hydra::row_copy_plan(row16);
  const int64_t most = hydra::row_copy_most_rows(args.rows);
  hipError_t err = hipSuccess;
  for (int64_t at = 0; at < rows && err == hipSuccess; at += most) {
    const int64_t here = rows - at < most ? rows - at : most;
    args.rows.first_row = (int32_t)at;
    args.rows.rows = (int32_t)here;
    err = launch(args.rows.waves != 0 ? kilobytes : others, dim3((unsigned)hydra::row_copy_workgroups(args.rows, here)), dim3(hydra::kRowCopyThreads), stream, args);
  }
  return err;
}

// Compute units of the current device (0 if the runtime cannot tell).  Looked up on every call:
// the library keeps no state, and the attribute query does not touch the device.
unsigned compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 0;
  return (unsigned)n;
}

// One launch: the persistent workgroups drain the work list (an item whose exponentials leave the
// fast path's range is redone on the spot, by the same workgroup, with the careful routine).
template <int D>
hipError_t launch_attn(bool causal, const hydra::AttnArgs& args, unsigned compute_units, int workgroups_per_cu, hipStream_t stream) {
  // two or three persistent workgroups per compute unit (each takes its share of registers and LDS):
  // while one is loading Q, storing O or between key blocks, the others' matrix work fills the SIMDs.
  // A caller that runs another kernel beside this one asks for fewer (workgroups_per_cu > 0); any number
  // of workgroups drains the queues.
  const unsigned per_cu = workgroups_per_cu > 0 && workgroups_per_cu < hydra::kWorkgroupsPerCu<D> ? (unsigned)workgroups_per_cu
                                                                                                  : (unsigned)hydra::kWorkgroupsPerCu<D>;
  const unsigned grid = per_cu * compute_units;
  return causal ? launch(hydra::attn_fwd_kernel<D, true>, dim3(grid), dim3(256), stream, args)
                : launch(hydra::attn_fwd_kernel<D, false>, dim3(grid), dim3(256), stream, args);
}

// How a batch of up to `capacity` items runs: one workgroup per item up to kDirectRounds rounds of the chip's workgroup
// slots, and up to kListFreeRounds without a work list if the call would have to build it (attn_fwd_direct_kernel).
// us per call with persistent workgroups and so: 4 images of 577 tokens 27.5 -> 13.9, 14 images 45.1 -> 31.9, 32 images 71 -> 63.
// us per call without a list and with one built first, by rounds: 16 heads of 64, 14 images of 577 tokens (1.5 rounds) 32.8 and 35.9, 26
// (2.7) 53.6 and 56.4, 30 (3.1) 60.3 and 62.9, 34 (3.5) 68.5 and 69.6, 38 (4.0) 77.4 and 76.9; 16 heads of 80, 17 000 tokens in images
// of 256 .. 4096 (2.9) 194.1 and 194.8, 19 000 (3.3) 204.3 and 207.6, 21 000 (3.6) 223.1 and 222.1, 23 000 (4.0) 243.3 and 243.5;
// 28 / 4 heads of 128, 6 requests (1.5) 28.2 and 30.6, 10 (2.5) 41.6 and 41.3, 14 (3.4) 54.1 and 53.6, 18 (4.3) 66.3 and 65.7; 32 / 32
// heads of 128, 2 requests of 700 tokens (0.8) 18.4 and 21.7, 3 (1.1) 27.4 and 26.2, 4 (1.5) 33.8 and 32.3, 5 (1.9) 38.2 and 39.6.
constexpr size_t kDirectRounds = 6, kListFreeRounds = 4;
bool within_rounds(size_t rounds, int32_t head_dim, size_t capacity, unsigned compute_units) {
  const unsigned per_cu = head_dim == 64 ? hydra::kDirectPerCu<64> : head_dim == 80 ? hydra::kDirectPerCu<80> : hydra::kDirectPerCu<128>;
  return capacity <= rounds * per_cu * compute_units;
}
// (head_dim 80 beyond that too: see kDirectPerCu.  Measured up to 640 000 items, 40 000 images of 16 tokens with 16 heads, 4782 us with
// persistent workgroups, 4136 so; longer lists than a million stay with those.)
bool direct_form(int32_t head_dim, size_t capacity, unsigned compute_units) {
  return within_rounds(kDirectRounds, head_dim, capacity, compute_units) || (head_dim == 80 && capacity <= (size_t)1 << 20);
}
bool list_free(int32_t batch, int32_t head_dim, size_t capacity, unsigned compute_units) {
  return batch <= hydra::kDirectSeqs && within_rounds(kListFreeRounds, head_dim, capacity, compute_units);
}
// Whether a batch at head_dim 80 has about four items of short sequences per compute unit: then two of its workgroups share a unit
// instead of three, which would leave the fourth alone with the unit's SIMDs.  Items are exact where all sequences have max_seqlen
// tokens, and an average otherwise (half a wave tile and three eighths of an item of every sequence are padding).
// us with three and with two, causal: 28 / 4 heads, sequences of 272 tokens, 832 items 17.9 and 17.2, 896 19.7 and 17.3, 960 20.5 and 18.2;
// of 384, 840 20.7 and 19.3, 924 22.8 and 19.9; 16 heads, of 256, 800 21.9 and 22.0, 864 23.3 and 22.7, 992 26.9 and 23.1, 1056 27.1 and
// 27.4; of 64 .. 448, 896 23.0 and 20.4; of 384, 864 23.6 and 23.1, 1056 26.5 and 28.6 (8 heads).  Bidirectional, where the items differ less:
// 28 / 4 heads of 272, 832 21.9 and 22.7, 896 equal, 1024 24.0 and 23.2; 16 heads, of 64 .. 448, 896 26.9 and 24.9, 976 26.7 and 24.1;
// but of 384 tokens with 28 / 4 heads 924 25.0 and 26.2.
bool four_short_items(bool causal, int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, unsigned compute_units) {
  const float most_tokens = causal ? 400.0f : 300.0f, least_items = causal ? 3.15f : 3.3f;
  const float seqs = (float)batch, kv_heads = (float)n_kv_heads, units = (float)compute_units;
  if ((float)total_tokens > most_tokens * seqs) return false;
  const int32_t group = n_q_heads / n_kv_heads;
  float items = kv_heads * ((float)group * ((float)total_tokens / hydra::kWaveTileRows + 0.5f * seqs) / hydra::kWavesPerItem + 0.375f * seqs);
  if ((int64_t)max_seqlen * batch == total_tokens) items = kv_heads * seqs * (float)hydra::items_of_sequence(max_seqlen, group);
  return items > least_items * units && items <= 4.0f * units;
}
// (what the header tells callers of hydra_attn_varlen_fwd_shared about these workgroups' LDS, with 128 bytes for the kernel's own words)
template <int D>
constexpr bool shared_lds_within(int kilobytes) { return hydra::TileGeom<D, 2, hydra::DirectSource<2, 0>::kStageRows>::kLdsBytes + 128 <= kilobytes * 1024; }
static_assert(shared_lds_within<64>(67) && shared_lds_within<80>(92) && shared_lds_within<128>(131), "as the header says");
// listed: the items come from the work list, whose entries, four wave tiles or the rest of a sequence, the workgroups share.
template <int D, int TEAMS, int LOADERS>
hipError_t launch_direct(bool causal, const hydra::AttnArgs& args, bool listed, int32_t batch, int32_t total_tokens, int32_t n_kv_heads, bool two_per_unit, hipStream_t stream) {
  using Source = hydra::DirectSource<TEAMS, LOADERS>;
  const dim3 grid((unsigned)hydra::direct_workgroups(Source::kTiles, listed ? hydra::kWavesPerItem : Source::kTiles, batch, total_tokens, args.group, n_kv_heads));
  // (LDS that is asked for and not used, so that a third workgroup does not fit)
  constexpr size_t kThird = hydra::kLdsPerUnit / 3, kLds = hydra::TileGeom<D, TEAMS, Source::kStageRows>::kLdsBytes;
  const size_t pad = two_per_unit && kLds < kThird ? kThird - kLds : 0;
  return launch_lds(causal ? hydra::attn_fwd_direct_kernel<D, true, TEAMS, LOADERS> : hydra::attn_fwd_direct_kernel<D, false, TEAMS, LOADERS>, grid, dim3(Source::kThreads), pad,
                    stream, args, listed ? 0 : batch, n_kv_heads);
}

// Bytes of one partial result of the paged kernel's packed-rows form.
size_t paged_partial_bytes(int head_dim) { return (size_t)(2 * hydra::paged::kRows + hydra::paged::kRows * head_dim) * sizeof(float); }

// Workgroups per (request, KV head) pair over which the paged kernels split a context: of the two numbers that fill the
// chip's 256 compute units once (first) and twice (second) with the pairs' shares, 1 each where splitting does not pay.
// A function of the launch sizes alone: the workspace query and the launch both use it.
//   - One compute unit fetches at most 48 GB/s of a stream from HBM, whatever its waves keep in flight, so one workgroup
//     needs 2.7 us per 256 keys of a KV head (512 bytes each at head_dim 128), and the combine kernel costs 2.5 us: a
//     split pays from about 600 keys saved on.
//   - The keys per compute unit are what counts: 48 pairs of up to 3731 keys take 15.1 us in 5 shares (240 workgroups),
//     17.5 in 6 (288: some units get two shares), 15.8 in 10 (480).
//   - More than 256 pairs are not split: the extra workgroups and the merge cost more than the imbalance they remove.
struct PagedSplits {
  int once, twice;
};
PagedSplits paged_splits(int32_t batch, int32_t n_kv_heads, int32_t max_blocks_per_seq, int32_t block_size) {
  constexpr int64_t kUnits = 256, kSavedKeys = 600;
  const int64_t pairs = (int64_t)batch * n_kv_heads, keys = (int64_t)max_blocks_per_seq * block_size;
  auto fill = [&](int64_t layers) {
    int64_t n = layers * kUnits / pairs;
    if (n > hydra::paged::kMaxSplits) n = hydra::paged::kMaxSplits;
    return n < 2 || pairs > kUnits || keys - keys / n < kSavedKeys ? 1 : (int)n;
  };
  return {fill(1), fill(2)};
}
// The number of the two that leaves fewer keys to the busiest compute unit (the larger one only where it is 10 % fewer),
// as far as the workspace holds that many partial results.
// tile_wgs: workgroups for prefill chunks in the same batch.  Unless contexts are long, the kernel waits for the chunks'
// chains of key tiles, and a share on a chain's unit slows it down.  So beside chunks a context has one share per 512 keys, except on
// units that the chunks leave free, and nothing is split where the decode steps alone take more than half of the units.
// us, shares as without chunks and now: 20 decode steps of up to 800 keys and a chunk of 512 21.0 -> 15.1; 4 of up to 1000 and
// 3 chunks of 128 16.9 -> 12.6; 10 of up to 2500 and 4 of 512 55.5 -> 50.4; 30 of up to 2000 and 2 of 512 36.0 -> 31.5.  Split in
// two with 204 pairs 29.6 instead of 26.9; 4 of up to 2500 and a chunk of 60 in 4 shares 11.3 instead of 10.6 in 9.
// *least_log2: half tiles up to which a context is not cut further (share_plan).  Beside chunks 512 keys, as above; otherwise
// one half tile per wave, and more where shares are few and long anyway, since short contexts then only add to the merge
// (30 requests of 100 .. 1400 tokens in 2 shares: 14.4 us with 4 half tiles, 14.0 with 16).
int choose_splits(PagedSplits s, int64_t pairs, int64_t keys, int64_t tile_wgs, int32_t head_dim, size_t workspace_bytes, int32_t* least_log2) {
  // (beside chunks as many shares as were measured there)
  if (tile_wgs > 0) s = {s.once < 16 ? s.once : 16, s.twice < 16 ? s.twice : 16};
  auto layers = [&](int64_t n) { return (pairs * n + 255) / 256; };  // shares on the busiest unit, of 1 / n of a context
  int64_t n = layers(s.twice) * s.once * 10 < layers(s.once) * s.twice * 9 ? s.twice : s.once;
  int32_t beside_chunks = 0;
  if (tile_wgs > 0) {
    const int64_t free_units = (256 - tile_wgs) / pairs < s.once ? (256 - tile_wgs) / pairs : s.once;
    n = s.once > 1 ? (keys / 512 < s.twice ? keys / 512 : s.twice) : 1;
    if (n > 2 && free_units >= n) n = free_units;
    else beside_chunks = 4;
  }
  const int64_t fits = (int64_t)(workspace_bytes / (paged_partial_bytes(head_dim) * (size_t)pairs));
  if (n > fits) n = fits;
  if (n < 2) n = 1;
  const int64_t halves = (keys < 2048 ? keys : 2048) / 32 / n;
  *least_log2 = beside_chunks != 0 ? beside_chunks : halves < 8 ? 2 : halves < 16 ? 3 : 4;
  // No more than the longest context that the table describes can have: fewer empty workgroups, and a shorter merge.  (Where contexts
  // are cut stays the same.  Beside chunks the number has a say in where they go: left.)
  const int64_t most = ((keys + 31) / 32 + ((int64_t)1 << *least_log2) - 1) >> *least_log2;
  if (tile_wgs == 0 && n > most) n = most;
  return (int)n;
}

// Launches of attn_paged_fwd for one head dimension: the decode kernel when no request of the batch has more rows than
// its form takes, otherwise the kernel that holds all forms; then the merge of split contexts.
template <int D>
hipError_t launch_paged(const hydra::paged::PagedArgs& args, int32_t total_q, int32_t max_q_len, bool decode_only, unsigned rows_wgs, unsigned tile_wgs, hipStream_t s) {
  hipError_t err;
  bool launched = false;
  if constexpr (hydra::paged::kDecodeForm<D>) {
    if (decode_only) {
      const int64_t keys = (int64_t)args.max_blocks_per_seq << args.block_shift;
      const bool ordered = hydra::paged::decode_ordered(rows_wgs, args.n_splits, args.batch, keys);
      using hydra::paged::kDecodeMaxStreams, hydra::paged::kDecodeWaves, hydra::paged::attn_decode_kernel;
      constexpr int kFour = kDecodeWaves, kEight = kDecodeMaxStreams;
      const int streams = hydra::paged::decode_streams(rows_wgs, args.n_splits, keys), waves = hydra::paged::decode_waves(rows_wgs, streams, ordered);
      void (*kernel)(hydra::paged::PagedArgs) = attn_decode_kernel<D, false, kFour, kFour>;
      if (ordered) kernel = streams == kFour ? attn_decode_kernel<D, true, kFour, kFour> : waves == kFour ? attn_decode_kernel<D, true, kFour, kEight> : attn_decode_kernel<D, true, kEight, kEight>;
      else if (streams == kEight) kernel = attn_decode_kernel<D, false, kEight, kEight>;
      const dim3 grid = ordered ? dim3(rows_wgs) : dim3((unsigned)args.n_kv_heads, (unsigned)args.batch, (unsigned)args.n_splits);
      err = launch_lds(kernel, grid, dim3(64 * waves), streams * hydra::paged::kDecodeLdsPerWave<D>, s, args);
      launched = true;
    }
  }
  if (!launched) {
    unsigned grid = rows_wgs + tile_wgs;
    if constexpr (D != 80) {
      // (the pipeline asks for rows of a cache block that are whole load instructions, and for row numbers of 32 bits)
      const bool pipeline = (1 << args.block_shift) >= 1024 / (2 * D) && args.num_blocks <= (0x7fffffff >> args.block_shift);
      const hydra::rules::Hybrid batch{args.batch, total_q, max_q_len, args.group, args.n_kv_heads, args.n_splits, (int64_t)args.max_blocks_per_seq << args.block_shift};
      if (const hydra::rules::WideGrid g = hydra::rules::wide_grid(batch); tile_wgs > 0 && pipeline && g.use) {
        hydra::paged::PagedArgs wide_args = args;
        if (g.by_context) wide_args.order_keys = 0;
        err = launch(hydra::paged::attn_paged_kernel<D, true>, dim3((unsigned)(g.workgroups < grid + 16 ? g.workgroups : grid + 16)), dim3(512), s, wide_args);
        launched = true;
      }
    }
    if (!launched) {
      // (find_work deals out decode steps and chains over both layers of the chip, and may leave seven places of the first unused)
      if (tile_wgs > 0 && args.batch <= hydra::paged::kOrderedMost) grid = grid + 7 < 2 * hydra::paged::kUnits ? 2 * hydra::paged::kUnits : grid + 7;
      err = launch(hydra::paged::attn_paged_kernel<D, false>, dim3(grid), dim3(256), s, args);
    }
  }
  if (err == hipSuccess && args.n_splits > 1) {
    const int64_t rows = (int64_t)max_q_len * args.group;
    const int64_t pieces = (rows < hydra::paged::kRows ? rows : hydra::paged::kRows) * (D / 4);
    // (a merge with as little code as the number of shares allows: see the kernel)
    auto merge = [&](auto groups, auto each) {
      constexpr int kGroups = decltype(groups)::value, kPieces = hydra::paged::kCombinePieces<kGroups>;
      return launch(hydra::paged::attn_paged_combine_kernel<D, kGroups, decltype(each)::value>,
                    dim3((unsigned)args.n_kv_heads, (unsigned)args.batch, (unsigned)((pieces + kPieces - 1) / kPieces)),
                    dim3(hydra::paged::kCombineThreads<kGroups>), s, args);
    };
    using std::integral_constant;
    if (args.n_splits <= 2) err = merge(integral_constant<int, 1>{}, integral_constant<int, 2>{});
    else if (args.n_splits <= 4) err = merge(integral_constant<int, 1>{}, integral_constant<int, 4>{});
    else if (args.n_splits <= 16) err = merge(integral_constant<int, 4>{}, integral_constant<int, 4>{});
    else err = merge(integral_constant<int, 8>{}, integral_constant<int, 8>{});
  }
  return err;
}

}  // namespace

extern "C" {

size_t hydra_attn_workspace_bytes(int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads,
                                  int32_t head_dim) {
  if (batch < 0 || total_tokens < 0 || max_seqlen < 0 || n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0 ||
      !head_dim_supported(head_dim))
    return 0;
  return hydra::workspace_layout(batch, total_tokens, n_q_heads, n_kv_heads).total;
}

const char* hydra_status_string(int status) {
  switch (status) {
    case HYDRA_OK: return "ok";
    case HYDRA_ERR_INVALID_ARG: return "invalid argument";
    case HYDRA_ERR_UNSUPPORTED: return "unsupported configuration";
    case HYDRA_ERR_WORKSPACE: return "workspace missing or too small";
    case HYDRA_ERR_LAUNCH: return "kernel launch failed";
    default: return "unknown status";
  }
}

namespace {

// Argument checks shared by the three attention entry points.  `need_tensors` is false for the
// work-list builder, which touches only cu_seqlens and the workspace.
int check_attn_sizes(int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim) {
  if (batch < 0 || total_tokens < 0 || n_q_heads <= 0 || n_kv_heads <= 0) return HYDRA_ERR_INVALID_ARG;
  if (n_q_heads % n_kv_heads != 0) return HYDRA_ERR_INVALID_ARG;
  if (!head_dim_supported(head_dim)) return HYDRA_ERR_UNSUPPORTED;
  if (batch > 0 && total_tokens > 0 && max_seqlen < 1) return HYDRA_ERR_INVALID_ARG;
  // 32-bit byte offsets inside one sequence's K/V rows (buffer addressing in the attention kernel)
  // are checked by the callers that know the strides; 32-bit index arithmetic inside the prepass:
  if ((int64_t)n_q_heads * ((int64_t)total_tokens / hydra::kWaveTileRows + batch) > (int64_t)1 << 30) return HYDRA_ERR_UNSUPPORTED;
  return HYDRA_OK;
}

int check_workspace(const void* workspace, size_t workspace_bytes, const hydra::WorkspaceLayout& lay) {
  if (!workspace || workspace_bytes < lay.total || !aligned16(workspace)) return HYDRA_ERR_WORKSPACE;
  return HYDRA_OK;
}

}  // namespace

int hydra_attn_build_worklist(const int32_t* cu_seqlens, int32_t batch, int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads,
                              int32_t n_kv_heads, int32_t head_dim, int32_t causal, void* workspace, size_t workspace_bytes,
                              void* stream) {
  if (int rc = check_attn_sizes(batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim)) return rc;
  if (batch == 0 || total_tokens == 0) return HYDRA_OK;
  if (!cu_seqlens) return HYDRA_ERR_INVALID_ARG;
  const hydra::WorkspaceLayout lay = hydra::workspace_layout(batch, total_tokens, n_q_heads, n_kv_heads);
  if (int rc = check_workspace(workspace, workspace_bytes, lay)) return rc;

  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  hydra::WorkControl* ctrl = reinterpret_cast<hydra::WorkControl*>(ws);
  int32_t* sorted_seq = reinterpret_cast<int32_t*>(ws + lay.sorted_at);
  int32_t* queue_prefix = reinterpret_cast<int32_t*>(ws + lay.prefix_at);
  hydra::WorkItem* items = reinterpret_cast<hydra::WorkItem*>(ws + lay.items_at);
  const int group = n_q_heads / n_kv_heads;
  const int tail_items = hydra::tail_sort_items(group, head_dim);
  const dim3 grid(hydra::prepass_workgroups(lay.capacity)), block(hydra::kPrepassThreads);
  const hipError_t err =
      causal ? launch(hydra::build_worklist_kernel<true>, grid, block, s, cu_seqlens, batch, n_kv_heads, group, ctrl, sorted_seq, queue_prefix,
                      (int)lay.rows, items, (int)lay.capacity, tail_items)
             : launch(hydra::build_worklist_kernel<false>, grid, block, s, cu_seqlens, batch, n_kv_heads, group, ctrl, sorted_seq, queue_prefix,
                      (int)lay.rows, items, (int)lay.capacity, tail_items);
  return err == hipSuccess ? HYDRA_OK : HYDRA_ERR_LAUNCH;
}

namespace {

// Every host-side check of an attention call (sizes, pointers, strides, 32-bit addressing limits, the
// workspace, the device), shared by the entry points so that each of them has finished checking
// before its first launch.  *done is set when the call has nothing to do; *cus receives the number of
// compute units.
int validate_attn_call(const void* q, const void* k, const void* v, const void* out, int64_t q_token_stride, int64_t k_token_stride,
                       int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch, int32_t total_tokens, int32_t max_seqlen,
                       int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, float softmax_scale, const void* workspace,
                       size_t workspace_bytes, bool* done, unsigned* cus) {
  *done = false;
  if (int rc = check_attn_sizes(batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim)) return rc;
  if (!(softmax_scale >= 0.0f) || isinf(softmax_scale)) return HYDRA_ERR_INVALID_ARG;
  if (batch == 0 || total_tokens == 0) {
    *done = true;
    return HYDRA_OK;
  }
  if (!q || !k || !v || !out || !cu_seqlens) return HYDRA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(out)) return HYDRA_ERR_INVALID_ARG;
  if (q_token_stride < (int64_t)n_q_heads * head_dim || k_token_stride < (int64_t)n_kv_heads * head_dim ||
      v_token_stride < (int64_t)n_kv_heads * head_dim)
    return HYDRA_ERR_INVALID_ARG;
  if ((q_token_stride | k_token_stride | v_token_stride) & 7) return HYDRA_ERR_INVALID_ARG;
  {
    // the kernel addresses one sequence's K (or V) rows with 32-bit byte offsets
    const int64_t widest = k_token_stride > v_token_stride ? k_token_stride : v_token_stride;
    if (((int64_t)max_seqlen + 2 * hydra::kKvTileRows) * widest * 2 >= ((int64_t)1 << 31)) return HYDRA_ERR_UNSUPPORTED;
  }
  if (int rc = check_workspace(workspace, workspace_bytes, hydra::workspace_layout(batch, total_tokens, n_q_heads, n_kv_heads))) return rc;
  *cus = compute_units();
  if (*cus == 0) return HYDRA_ERR_LAUNCH;
  return HYDRA_OK;
}

// The attention launch; with_list: against a prebuilt work list; workgroups_per_cu == 0: the kernel's own number.
int launch_packed(const void* q, const void* k, const void* v, void* out, int64_t q_token_stride, int64_t k_token_stride,
                  int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch, int32_t total_tokens, int32_t max_seqlen,
                  int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int32_t causal, float softmax_scale, void* workspace,
                  size_t workspace_bytes, bool with_list, int32_t workgroups_per_cu, void* stream) {
  bool done = false;
  unsigned cus = 0;
  if (int rc = validate_attn_call(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                                  n_q_heads, n_kv_heads, head_dim, softmax_scale, workspace, workspace_bytes, &done, &cus))
    return rc;
  if (done) return HYDRA_OK;
  const hydra::WorkspaceLayout lay = hydra::workspace_layout(batch, total_tokens, n_q_heads, n_kv_heads);

  unsigned char* ws = static_cast<unsigned char*>(workspace);
  hydra::AttnArgs args;
  args.q = static_cast<const uint16_t*>(q);
  args.k = static_cast<const uint16_t*>(k);
  args.v = static_cast<const uint16_t*>(v);
  args.out = static_cast<uint16_t*>(out);
  args.q_stride = q_token_stride;
  args.k_stride = k_token_stride;
  args.v_stride = v_token_stride;
  args.cu_seqlens = cu_seqlens;
  args.items = reinterpret_cast<const hydra::WorkItem*>(ws + lay.items_at);
  args.ctrl = reinterpret_cast<hydra::WorkControl*>(ws);
  args.n_q_heads = n_q_heads;
  args.group = n_q_heads / n_kv_heads;
  // A scale of exactly 0 is replaced by a vanishing positive one: every visible key still gets
  // weight exp2(~0) = 1, while -inf (masked) times the scale stays -inf instead of becoming NaN.
  const float scale_log2 = softmax_scale * 1.44269504088896340736f;
  args.scale_log2 = scale_log2 > 1e-30f ? scale_log2 : 1e-30f;

  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t err;
  auto launch_for = [&](auto d) {
    constexpr int D = decltype(d)::value;
    const bool is_causal = causal != 0;
    if (hydra::rules::halved_items(D, batch, total_tokens, n_q_heads, n_kv_heads, cus)) {
      return workgroups_per_cu == 0 ? launch_direct<D, 2, 2>(is_causal, args, with_list, batch, total_tokens, n_kv_heads, false, s)
                                    : launch_direct<D, 2, 0>(is_causal, args, with_list, batch, total_tokens, n_kv_heads, false, s);
    }
    if (workgroups_per_cu != 0 || (with_list && !direct_form(head_dim, lay.capacity, cus))) return launch_attn<D>(is_causal, args, cus, workgroups_per_cu, s);
    if (hydra::rules::loading_waves(is_causal, batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, cus))
      return launch_direct<D, 1, 4>(is_causal, args, with_list, batch, total_tokens, n_kv_heads, false, s);
    const bool two = D == 80 && four_short_items(is_causal, batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, cus);
    return launch_direct<D, 1, 0>(is_causal, args, with_list, batch, total_tokens, n_kv_heads, two, s);
  };
  switch (head_dim) {
    case 64: err = launch_for(std::integral_constant<int, 64>{}); break;
    case 80: err = launch_for(std::integral_constant<int, 80>{}); break;
    default: err = launch_for(std::integral_constant<int, 128>{}); break;
  }
  return err == hipSuccess ? HYDRA_OK : HYDRA_ERR_LAUNCH;
}

}  // namespace

int hydra_attn_varlen_fwd_prebuilt(const void* q, const void* k, const void* v, void* out, int64_t q_token_stride,
                                   int64_t k_token_stride, int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch,
                                   int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                   int32_t causal, float softmax_scale, void* workspace, size_t workspace_bytes, void* stream) {
  return launch_packed(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                       n_q_heads, n_kv_heads, head_dim, causal, softmax_scale, workspace, workspace_bytes, true, 0, stream);
}

int hydra_attn_varlen_fwd_shared(const void* q, const void* k, const void* v, void* out, int64_t q_token_stride,
                                 int64_t k_token_stride, int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch,
                                 int32_t total_tokens, int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                                 int32_t causal, float softmax_scale, void* workspace, size_t workspace_bytes,
                                 int32_t workgroups_per_cu, void* stream) {
  if (workgroups_per_cu < 1) return HYDRA_ERR_INVALID_ARG;
  return launch_packed(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                       n_q_heads, n_kv_heads, head_dim, causal, softmax_scale, workspace, workspace_bytes, true, workgroups_per_cu, stream);
}

int hydra_attn_varlen_fwd(const void* q, const void* k, const void* v, void* out, int64_t q_token_stride, int64_t k_token_stride,
                          int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch, int32_t total_tokens, int32_t max_seqlen,
                          int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int32_t causal, float softmax_scale, void* workspace,
                          size_t workspace_bytes, void* stream) {
  // every check of both halves runs before the first launch, so that an error never leaves half the work enqueued
  bool done = false;
  unsigned cus = 0;
  if (int rc = validate_attn_call(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                                  n_q_heads, n_kv_heads, head_dim, softmax_scale, workspace, workspace_bytes, &done, &cus))
    return rc;
  if (done) return HYDRA_OK;

  const bool with_list = !list_free(batch, head_dim, hydra::item_capacity(batch, total_tokens, n_q_heads, n_kv_heads), cus);
  if (with_list) {
    if (int rc = hydra_attn_build_worklist(cu_seqlens, batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim, causal, workspace,
                                           workspace_bytes, stream))
      return rc;
  }
  return launch_packed(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen, n_q_heads,
                       n_kv_heads, head_dim, causal, softmax_scale, workspace, workspace_bytes, with_list, 0, stream);
}

}  // extern "C"

namespace {

// Work-list memory of hydra_attn_varlen_fwd_static: one array per device, living in the code
// object's data segment, so that a caller that may not allocate needs no workspace of its own.
constexpr size_t kStaticScratchBytes = HYDRA_ATTN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Device address of `scratch` on the current device.  In host code the array's name is only a
// handle for the runtime, so the address is asked for once per device (with that device current)
// and kept; every use below goes through this pointer.
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

int static_scratch(void** ptr) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return HYDRA_ERR_LAUNCH;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return HYDRA_ERR_LAUNCH;
    g_scratch_ptr[dev].store(p, std::memory_order_release);  // (two first callers get the same address)
  }
  *ptr = p;
  return HYDRA_OK;
}

}  // namespace

extern "C" {

int hydra_attn_varlen_fwd_static(const void* q, const void* k, const void* v, void* out, int64_t q_token_stride, int64_t k_token_stride,
                                 int64_t v_token_stride, const int32_t* cu_seqlens, int32_t batch, int32_t total_tokens,
                                 int32_t max_seqlen, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int32_t causal,
                                 float softmax_scale, void* stream) {
  // sizes first: the work list of this call has to fit the static array
  if (int rc = check_attn_sizes(batch, total_tokens, max_seqlen, n_q_heads, n_kv_heads, head_dim)) return rc;
  if (batch == 0 || total_tokens == 0)  // nothing to launch; the remaining argument checks are the plain call's
    return hydra_attn_varlen_fwd(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                                 n_q_heads, n_kv_heads, head_dim, causal, softmax_scale, nullptr, 0, stream);
  if (hydra::workspace_layout(batch, total_tokens, n_q_heads, n_kv_heads).total > kStaticScratchBytes) return HYDRA_ERR_WORKSPACE;
  void* ws = nullptr;
  if (int rc = static_scratch(&ws)) return rc;
  // Where a work list is used, the prepass rewrites every word of it, of the counters and of the flags that the attention
  // kernels read, and otherwise nothing is read, so whatever the previous call left in the array does not matter.
  return hydra_attn_varlen_fwd(q, k, v, out, q_token_stride, k_token_stride, v_token_stride, cu_seqlens, batch, total_tokens, max_seqlen,
                               n_q_heads, n_kv_heads, head_dim, causal, softmax_scale, ws, kStaticScratchBytes, stream);
}

int hydra_attn_paged_fwd(const void* q, void* out, int64_t q_token_stride, const void* k_cache, const void* v_cache,
                         const int32_t* block_tables, int32_t max_blocks_per_seq, const int32_t* cu_seqlens_q, const int32_t* kv_lens,
                         int32_t batch, int32_t total_q, int32_t max_q_len, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                         int32_t block_size, int64_t num_blocks, float softmax_scale, void* workspace, size_t workspace_bytes,
                         void* stream) {
  if (batch < 0 || total_q < 0 || n_q_heads <= 0 || n_kv_heads <= 0 || n_q_heads % n_kv_heads != 0) return HYDRA_ERR_INVALID_ARG;
  if (!head_dim_supported(head_dim)) return HYDRA_ERR_UNSUPPORTED;
  if (block_size < 1 || (block_size & (block_size - 1)) != 0) return HYDRA_ERR_UNSUPPORTED;
  if (!(softmax_scale >= 0.0f) || isinf(softmax_scale)) return HYDRA_ERR_INVALID_ARG;
  if (batch == 0 || total_q == 0) return HYDRA_OK;
  if (max_q_len < 1 || max_blocks_per_seq < 1 || num_blocks < 1) return HYDRA_ERR_INVALID_ARG;
  if (!q || !out || !k_cache || !v_cache || !block_tables || !cu_seqlens_q || !kv_lens) return HYDRA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(out) || !aligned16(k_cache) || !aligned16(v_cache)) return HYDRA_ERR_INVALID_ARG;
  if (q_token_stride < (int64_t)n_q_heads * head_dim || (q_token_stride & 7)) return HYDRA_ERR_INVALID_ARG;
  if (batch > 65535 || n_kv_heads > 65535 || num_blocks * block_size > (int64_t)0x7fffffff) return HYDRA_ERR_UNSUPPORTED;
  if ((int64_t)max_blocks_per_seq * block_size > (int64_t)1 << 30) return HYDRA_ERR_UNSUPPORTED;
  if (workspace_bytes > 0 && (!workspace || !aligned16(workspace))) return HYDRA_ERR_WORKSPACE;

  hydra::paged::PagedArgs args;
  args.q = static_cast<const uint16_t*>(q);
  args.out = static_cast<uint16_t*>(out);
  args.q_stride = q_token_stride;
  args.k_cache = static_cast<const uint16_t*>(k_cache);
  args.v_cache = static_cast<const uint16_t*>(v_cache);
  args.block_tables = block_tables;
  args.cu_seqlens_q = cu_seqlens_q;
  args.kv_lens = kv_lens;
  args.max_blocks_per_seq = max_blocks_per_seq;
  args.num_blocks = (int32_t)num_blocks;
  int shift = 0;
  while ((1 << shift) < block_size) ++shift;
  args.block_shift = shift;
  args.n_q_heads = n_q_heads;
  args.n_kv_heads = n_kv_heads;
  args.group = n_q_heads / n_kv_heads;
  const float scale_log2 = softmax_scale * 1.44269504088896340736f;
  args.scale_log2 = scale_log2 > 1e-30f ? scale_log2 : 1e-30f;  // (see hydra_attn_varlen_fwd_prebuilt)

  const int64_t tok_tiles = ((int64_t)max_q_len + hydra::paged::kRows - 1) / hydra::paged::kRows;
  int64_t groups = (tok_tiles * args.group + hydra::paged::kWavesPerGroup - 1) / hydra::paged::kWavesPerGroup;
  if ((int64_t)max_q_len * args.group <= hydra::paged::kRows) groups = 0;  // every request takes the packed-rows form
  args.partials = static_cast<float*>(workspace);
  args.batch = batch;
  // Workgroups of the wave-tile form: one per group of four wave tiles and KV head.  The request lengths are
  // on the device, so this is an upper bound from the total: a request of q new tokens has at most
  // (q / 32 + 1) * group / 4 + 1 groups.
  int64_t tile_wgs = 0;
  if (groups > 0) tile_wgs = (((int64_t)total_q / hydra::paged::kRows + batch) * args.group / hydra::paged::kWavesPerGroup + batch) * n_kv_heads;
  const int splits = choose_splits(paged_splits(batch, n_kv_heads, max_blocks_per_seq, block_size), (int64_t)batch * n_kv_heads,
                                   (int64_t)max_blocks_per_seq * block_size, tile_wgs, head_dim, workspace_bytes, &args.least_log2);
  args.n_splits = splits;
  const int64_t rows_wgs = (int64_t)batch * n_kv_heads * splits;
  if (tile_wgs + rows_wgs > (int64_t)0x7fffff00) return HYDRA_ERR_UNSUPPORTED;
  // The launch needs fewer: a request of this form has more than kRows rows, which bounds how many there are (where contexts are
  // cut is part of the result and stays with the number above).  Each of the others would look for its group in vain behind the
  // last one: 248 decode steps of 19 .. 194 tokens and a chunk of 21, 28 / 4 heads of 128, 22.6 -> 16.0 us.
  if (groups > 0) {
    const int64_t least_q = hydra::paged::kRows / args.group + 1, most_chunks = total_q / least_q < batch ? total_q / least_q : batch;
    tile_wgs = (((int64_t)total_q / hydra::paged::kRows + most_chunks) * args.group / hydra::paged::kWavesPerGroup + most_chunks) * n_kv_heads;
  }
  args.n_tile_wgs = (int32_t)tile_wgs;
  args.order_keys = hydra::paged::order_keys(batch, (int64_t)batch * n_kv_heads, (int64_t)max_blocks_per_seq * block_size, head_dim, tile_wgs);
  const bool decode_only = (int64_t)max_q_len * args.group <= hydra::paged::kDecodeRows && block_size >= hydra::paged::kDecodeMinBlock;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t err;
  switch (head_dim) {
    case 64: err = launch_paged<64>(args, total_q, max_q_len, decode_only, (unsigned)rows_wgs, (unsigned)tile_wgs, s); break;
    case 80: err = launch_paged<80>(args, total_q, max_q_len, decode_only, (unsigned)rows_wgs, (unsigned)tile_wgs, s); break;
    default: err = launch_paged<128>(args, total_q, max_q_len, decode_only, (unsigned)rows_wgs, (unsigned)tile_wgs, s); break;
  }
  return err == hipSuccess ? HYDRA_OK : HYDRA_ERR_LAUNCH;
}

size_t hydra_attn_paged_workspace_bytes(int32_t batch, int32_t n_kv_heads, int32_t head_dim, int32_t max_blocks_per_seq, int32_t block_size) {
  if (batch <= 0 || n_kv_heads <= 0 || !head_dim_supported(head_dim) || max_blocks_per_seq < 1 || block_size < 1) return 0;
  const PagedSplits splits = paged_splits(batch, n_kv_heads, max_blocks_per_seq, block_size);
  return splits.twice > 1 ? paged_partial_bytes(head_dim) * (size_t)splits.twice * (size_t)batch * (size_t)n_kv_heads : 0;
}

int hydra_kv_cache_write(const void* k, const void* v, int64_t k_token_stride, int64_t v_token_stride, void* k_cache, void* v_cache,
                         const int64_t* slot_mapping, int32_t total_tokens, int32_t n_kv_heads, int32_t head_dim, int32_t block_size,
                         int64_t num_blocks, void* stream) {
  if (total_tokens < 0 || n_kv_heads <= 0 || head_dim <= 0 || block_size <= 0 || num_blocks < 0) return HYDRA_ERR_INVALID_ARG;
  const int64_t row = (int64_t)n_kv_heads * head_dim;
  if (row % 8 != 0) return HYDRA_ERR_UNSUPPORTED;
  if (row > ((int64_t)1 << 24)) return HYDRA_ERR_UNSUPPORTED;
  if (total_tokens == 0) return HYDRA_OK;
  if (!k || !v || !k_cache || !v_cache || !slot_mapping) return HYDRA_ERR_INVALID_ARG;
  if (!aligned16(k) || !aligned16(v) || !aligned16(k_cache) || !aligned16(v_cache)) return HYDRA_ERR_INVALID_ARG;
  if (k_token_stride < row || v_token_stride < row || ((k_token_stride | v_token_stride) & 7)) return HYDRA_ERR_INVALID_ARG;

  hydra::KvWriteArgs args;
  args.k = static_cast<const hydra::piece_t*>(k);
  args.v = static_cast<const hydra::piece_t*>(v);
  args.k_cache = static_cast<hydra::piece_t*>(k_cache);
  args.v_cache = static_cast<hydra::piece_t*>(v_cache);
  args.slot_mapping = slot_mapping;
  args.k_stride16 = k_token_stride / 8;
  args.v_stride16 = v_token_stride / 8;
  const hipError_t err = launch_row_copy(hydra::kv_cache_write_kernel<true>, hydra::kv_cache_write_kernel<false>, args, total_tokens, (int32_t)(row / 8), static_cast<hipStream_t>(stream));
  return err == hipSuccess ? HYDRA_OK : HYDRA_ERR_LAUNCH;
}

namespace {

// Shared by the two image-cache calls: `packed` is the caller's row-major buffer (source of the write,
// destination of the gather).
int launch_page_cache(bool gather, const void* packed, int64_t packed_row_stride, const void* cache, const int64_t* slot_mapping,
                      int32_t n_rows, int32_t row_elems, int64_t num_slots, void* stream) {
  if (n_rows < 0 || row_elems <= 0 || num_slots < 0) return HYDRA_ERR_INVALID_ARG;
  if (row_elems % 8 != 0 || row_elems > (1 << 24)) return HYDRA_ERR_UNSUPPORTED;
  if (n_rows == 0) return HYDRA_OK;
  if (!packed || !cache || !slot_mapping) return HYDRA_ERR_INVALID_ARG;
  if (!aligned16(packed) || !aligned16(cache)) return HYDRA_ERR_INVALID_ARG;
  if (packed_row_stride < row_elems || (packed_row_stride & 7)) return HYDRA_ERR_INVALID_ARG;
  hydra::PageCacheArgs args;
  args.slot_mapping = slot_mapping;
  args.packed_stride16 = packed_row_stride / 8;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t err;
  if (gather) {
    args.src = static_cast<const hydra::piece_t*>(cache);
    args.dst = static_cast<hydra::piece_t*>(const_cast<void*>(packed));
    err = launch_row_copy(hydra::page_cache_kernel<true, true>, hydra::page_cache_kernel<true, false>, args, n_rows, row_elems / 8, s);
  } else {
    args.src = static_cast<const hydra::piece_t*>(packed);
    args.dst = static_cast<hydra::piece_t*>(const_cast<void*>(cache));
    err = launch_row_copy(hydra::page_cache_kernel<false, true>, hydra::page_cache_kernel<false, false>, args, n_rows, row_elems / 8, s);
  }
  return err == hipSuccess ? HYDRA_OK : HYDRA_ERR_LAUNCH;
}

}  // namespace

int hydra_page_cache_write(const void* rows, int64_t row_stride, void* cache, const int64_t* slot_mapping, int32_t n_rows, int32_t row_elems,
                           int64_t num_slots, void* stream) {
  return launch_page_cache(false, rows, row_stride, cache, slot_mapping, n_rows, row_elems, num_slots, stream);
}

int hydra_page_cache_gather(const void* cache, const int64_t* slot_mapping, void* rows, int64_t row_stride, int32_t n_rows, int32_t row_elems,
                            int64_t num_slots, void* stream) {
  return launch_page_cache(true, rows, row_stride, cache, slot_mapping, n_rows, row_elems, num_slots, stream);
}

}  // extern "C"
