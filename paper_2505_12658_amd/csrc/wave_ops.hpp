// Operations over the lanes of a wave.
#pragma once
#include <hip/hip_runtime.h>

namespace hydra {

#if defined(__HIP_DEVICE_COMPILE__)
// Sum over this lane and the lanes before it (data-parallel primitives: shifts inside the rows of 16 lanes, then the
// rows' totals handed on; a seventh of the latency of the six LDS permutes that a shuffle would take).
__device__ __forceinline__ int wave_scan_add(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return x;
}

// Sum over the lanes with the same number modulo 8 (rotation inside the rows of 16 lanes, then swaps of rows and of halves).
__device__ __forceinline__ int sum_of_columns(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false);
  int a = x, b = x;
  asm volatile("s_nop 3\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 3" : "+v"(a), "+v"(b));
  x = a + b;
  a = x;
  b = x;
  asm volatile("s_nop 3\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 3" : "+v"(a), "+v"(b));
  return a + b;
}
#endif  // __HIP_DEVICE_COMPILE__

}  // namespace hydra
