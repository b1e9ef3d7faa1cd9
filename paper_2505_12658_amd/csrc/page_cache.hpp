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
  RowCopyPlan rows;
};

// GATHER == false: cache[slot[t]] = packed[t];  GATHER == true: packed[t] = cache[slot[t]].
// KILOBYTES: the rows are whole kilobytes (rows.waves != 0).
template <bool GATHER, bool KILOBYTES>
__global__ __launch_bounds__(kRowCopyThreads) void page_cache_kernel(const PageCacheArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  int64_t t, slot;
  int32_t p;
  if (!piece_of_lane<KILOBYTES>(a.rows, a.slot_mapping, t, slot, p) || slot < 0) return;
  // Stores are plain, since what is written is read by the next kernel.  Rows of whole kilobytes are loaded non-temporally
  // (nothing here is read twice): 14 014 rows of 7 KB into the cache and back 66.3 us, with plain loads 72.1.  Other rows
  // end inside cache lines that the lanes of the next row read too: 50 000 rows of 1440 bytes 47.2 us with plain loads, 60.9
  // with non-temporal ones.
  const piece_t* src = a.src + (GATHER ? slot * a.rows.row16 : t * a.packed_stride16) + p;
  const piece_t x = KILOBYTES ? __builtin_nontemporal_load(src) : *src;
  a.dst[(GATHER ? t * a.packed_stride16 : slot * a.rows.row16) + p] = x;
#else
  (void)a;
#endif
}

}  // namespace hydra
