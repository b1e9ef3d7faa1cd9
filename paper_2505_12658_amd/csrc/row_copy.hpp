// What the two row-copy kernels (KV scatter, image cache) share: which wave moves which part of which row.
//
// One wave per kilobyte of a row (64 pieces of 16 bytes), row after row.  What bounds these kernels is HBM when there are
// many rows and latency when there are few, so a wave does one thing: the row, and with it the slot, is the same for all
// its lanes (the slot comes through the scalar cache), and its loads and stores are whole 128-byte lines.  One thread per
// piece with a 64-bit division of its own, over at most 8192 workgroups and the rest in a loop, was the first version:
// 14 014 rows of 7 KB into the image cache and back 72.7 -> 64.8 us (402 MB); 2, 4 or 8 pieces per lane 67.1, 70.0, 69.0.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hydra {

constexpr int kRowCopyThreads = 256;
typedef unsigned int piece_t __attribute__((ext_vector_type(4)));  // 16 bytes

constexpr int64_t kRowCopyMostWorkgroups = 1 << 23;  // per launch (a grid has at most 2^32 threads)

inline int32_t runs_of_row(int32_t row16) { return (row16 + 63) / 64; }  // waves per row
inline int64_t row_copy_workgroups(int32_t rows, int32_t row16) { return ((int64_t)rows * runs_of_row(row16) + kRowCopyThreads / 64 - 1) / (kRowCopyThreads / 64); }

#if defined(__HIP_DEVICE_COMPILE__)
// This wave's row and this lane's piece of it; false where there is none.
__device__ __forceinline__ bool piece_of_lane(int32_t rows, int32_t row16, int32_t runs, int64_t first_wg, int32_t& row, int32_t& piece) {
  const int64_t u = (first_wg + blockIdx.x) * (kRowCopyThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = runs == 1 ? u : (u >> 32 ? u / runs : (int64_t)((uint32_t)u / (uint32_t)runs));
  row = (int32_t)t;
  piece = (int32_t)(u - t * runs) * 64 + (threadIdx.x & 63);
  return t < rows && piece < row16;
}
__device__ __forceinline__ int64_t slot_of(const int64_t* slot_mapping, int32_t row) {
  return ((const __attribute__((address_space(4))) int64_t*)(uintptr_t)slot_mapping)[row];
}
#endif

}  // namespace hydra
