// Paged KV-cache scatter: K/V rows of the packed prefill batch -> cache[slot_mapping[t]].
// Pure data movement: both sides are whole rows although consecutive tokens land in unrelated pages (block size 16,
// Section 5.1 of the paper).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "row_copy.hpp"

namespace hydra {

struct KvWriteArgs {
  const piece_t* k;
  const piece_t* v;
  piece_t* k_cache;
  piece_t* v_cache;
  const int64_t* slot_mapping;
  int64_t k_stride16, v_stride16;  // token strides in 16-byte units
  RowCopyPlan rows;                // one row per token, n_kv_heads * head_dim elements
};

// Non-temporal on both sides: the rows are not read again here, and the cache lines are written whole; plain stores made
// the LLaVA prefill pass 168 -> 183 us.  The compiler puts the row loads behind the test of the slot, one round trip to
// memory later; held ahead of it, for launches that fit the chip at once, they won 0.0 - 0.4 us of passes of 11 - 60 us
// (4 decode steps 10.9 -> 10.8, hybrid batch 60.6 -> 60.2), too little for a second path.
template <bool KILOBYTES>  // the rows are whole kilobytes (rows.waves != 0)
__global__ __launch_bounds__(kRowCopyThreads) void kv_cache_write_kernel(const KvWriteArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  int64_t t, slot;
  int32_t p;
  if (!piece_of_lane<KILOBYTES>(a.rows, a.slot_mapping, t, slot, p)) return;
  const piece_t k = __builtin_nontemporal_load(a.k + t * a.k_stride16 + p);
  const piece_t v = __builtin_nontemporal_load(a.v + t * a.v_stride16 + p);
  if (slot < 0) return;
  __builtin_nontemporal_store(k, a.k_cache + slot * a.rows.row16 + p);
  __builtin_nontemporal_store(v, a.v_cache + slot * a.rows.row16 + p);
#else
  (void)a;
#endif
}

}  // namespace hydra
