// What the two row-copy kernels (KV scatter, image cache) share: which lane moves which 16-byte piece of which row.
//
// What bounds these kernels is HBM when there are many rows and latency when there are few.
// Rows of whole kilobytes (64 pieces): one wave per kilobyte, row after row.  The row, and with it the slot, is the same
// for all lanes of a wave (the slot comes through the scalar cache), and its loads and stores are whole 128-byte lines.
// Other rows would leave lanes of that wave without work (a row of one KV head of 64 has 8 pieces): their pieces are dealt
// to the lanes one after the other, rows end to end, and a lane asks for its own slot.
// us, one wave per kilobyte against end to end: KV scatter of 100 000 tokens with one KV head of 64 18.7 and 8.8, of 128 25.0
// and 18.2; 4000 tokens with 9 heads of 80 (90 pieces) 5.4 and 4.9; image cache, 50 000 rows of 16 bytes 6.2 and 2.7; rows
// of 7 KB 131 and 134, of 1 KB the same.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hydra {

constexpr int kRowCopyThreads = 256;
typedef unsigned int piece_t __attribute__((ext_vector_type(4)));  // 16 bytes

constexpr int64_t kRowCopyMostLanes = (int64_t)1 << 31;  // per launch (a grid has at most 2^32 threads; see row_of_unit)

// One launch: rows first_row .. first_row + rows - 1.
struct RowCopyPlan {
  int32_t first_row, rows;
  int32_t row16;      // 16-byte pieces per row
  int32_t waves;      // waves per row; 0: pieces end to end
  uint32_t magic;     // division by row16, see row_of_unit
  int32_t shift;
};

inline RowCopyPlan row_copy_plan(int32_t row16) {
  RowCopyPlan p = {};
  p.row16 = row16;
  p.waves = row16 % 64 == 0 ? row16 / 64 : 0;
  int log2 = 0;
  while ((1 << log2) < row16) ++log2;
  p.shift = 31 + log2;
  p.magic = (uint32_t)((((uint64_t)1 << p.shift) + row16 - 1) / row16);  // (2^31 .. 2^32 - 1)
  return p;
}
// Rows of one launch at most, and the workgroups for `rows` of them.
inline int64_t row_copy_most_rows(const RowCopyPlan& p) { return kRowCopyMostLanes / p.row16; }
inline int64_t row_copy_workgroups(const RowCopyPlan& p, int64_t rows) { return (rows * p.row16 + kRowCopyThreads - 1) / kRowCopyThreads; }

#if defined(__HIP_DEVICE_COMPILE__)
// u / row16, exact for u < 2^31: magic is 2^shift / row16 rounded up, and u times what that adds, less than
// row16 <= 2^(shift - 31) of 2^shift, stays below one part in row16.
__device__ __forceinline__ uint32_t row_of_unit(const RowCopyPlan& p, uint32_t u) { return (uint32_t)(((uint64_t)u * p.magic) >> p.shift); }

// This lane's row, the row's slot, and this lane's piece of it; false where there is none.  KILOBYTES: whether p.waves != 0
// (known to the compiler, so that row and slot stay in scalar registers).
template <bool KILOBYTES>
__device__ __forceinline__ bool piece_of_lane(const RowCopyPlan& p, const int64_t* slot_mapping, int64_t& row, int64_t& slot, int32_t& piece) {
  if constexpr (KILOBYTES) {
    const uint32_t u = blockIdx.x * (kRowCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (not row_of_unit: with its few instructions the waves ask for memory closer together, and 14 014 rows of 7 KB through the
    // image cache and back took 64.9 us instead of 64.4)
    const uint32_t t = p.waves == 1 ? u : u / (uint32_t)p.waves;
    if (t >= (uint32_t)p.rows) return false;
    piece = (int32_t)((u - t * p.waves) * 64 + (threadIdx.x & 63));
    row = (int64_t)p.first_row + t;
    slot = ((const __attribute__((address_space(4))) int64_t*)(uintptr_t)slot_mapping)[row];
  } else {
    const uint32_t u = blockIdx.x * kRowCopyThreads + threadIdx.x;
    const uint32_t t = row_of_unit(p, u);
    if (t >= (uint32_t)p.rows) return false;
    piece = (int32_t)(u - t * p.row16);
    row = (int64_t)p.first_row + t;
    slot = slot_mapping[row];
  }
  return true;
}
#endif

}  // namespace hydra
