// What a wavefront does by itself: waits for its memory operations, sums over its 64 lanes.
#pragma once
#include <hip/hip_runtime.h>

// until at most N of its vector memory loads are in flight
#define HMI_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 0xF) | (((N) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
// until its LDS operations (and scalar loads) are done
#define HMI_WAIT_LGKMCNT0() __builtin_amdgcn_s_waitcnt(0xC07F)
// What the wavefronts pass on through LDS before a barrier; direct-to-LDS copies are waited for where their rows are due
// (__syncthreads would wait for all of them, and for the stores, at the first barrier behind them).
#define HMI_BARRIER()                                                                              \
  {                                                                                                \
    asm volatile("" ::: "memory");                                                                 \
    HMI_WAIT_LGKMCNT0();                                                                           \
    __builtin_amdgcn_s_barrier();                                                                  \
    asm volatile("" ::: "memory");                                                                 \
  }

namespace hmi {

// Sum over the lanes, in every lane.  The tree of a butterfly of shuffles (lanes 32 apart first, neighbours last), to the bit,
// without its trips through the LDS crossbar: halves and rows of 16 change places in registers, and inside a row a rotation by
// 8, 4, 2, 1 brings each lane the value of lane i ^ 8, 4, 2, 1, since the partial sums repeat with that period.  Two rows' mean and
// variance 0.75 -> 0.25 us.
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

// Inclusive prefix sum over the 64 lanes: inside rows of 16 by row shifts, then across rows by row broadcasts (six
// additions with their operand moved on the way, where a shuffle is a trip through the LDS crossbar).
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

}  // namespace hmi
