// Paged image cache: rows of the vision encoder's output -> cache pages, and back.
//
// The paper keeps the encoder's image tokens in an image cache that is paged like the KV cache
// (Section 4.5; image-cache block size
// 576 in Section 5.1), so that a request can migrate between instances and repeated images can be
// reused.  Both directions are pure data movement.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "row_copy.hpp"

namespace hydra {

struct PageCacheArgs {
  const piece_t* src;           // write: packed rows, gather: the cache
  piece_t* dst;                 // write: the cache, gather: packed rows
  const int64_t* slot_mapping;  // one cache slot (page * page_rows + row in page) per packed row; < 0: row skipped
  int64_t packed_stride16;      // stride of the packed rows in 16-byte units
  int32_t n_rows;
  int32_t row16;                // 16-byte pieces per row
  int32_t runs;                 // runs_of_row(row16)
  int64_t first_wg;             // workgroups of the launches before this one
};

// GATHER == false: cache[slot[t]] = packed[t];  GATHER == true: packed[t] = cache[slot[t]].
template <bool GATHER>
__global__ __launch_bounds__(kRowCopyThreads) void page_cache_kernel(const PageCacheArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  int32_t t, p;
  if (!piece_of_lane(a.n_rows, a.row16, a.runs, a.first_wg, t, p)) return;
  const int64_t slot = slot_of(a.slot_mapping, t);
  if (slot < 0) return;
  // (non-temporal loads: nothing here is read twice; plain stores, since what is written is read by the next kernel:
  // image cache and back 64.8 us, both non-temporal 67.2, neither 69.3)
  const piece_t x = __builtin_nontemporal_load(a.src + (GATHER ? slot * a.row16 : t * a.packed_stride16) + p);
  a.dst[(GATHER ? t * a.packed_stride16 : slot * a.row16) + p] = x;
#else
  (void)a;
#endif
}

}  // namespace hydra
