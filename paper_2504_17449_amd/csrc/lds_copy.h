// Direct-to-LDS copies by buffer loads.  A global load to LDS counts among a wavefront's LDS operations too, out of order with
// its LDS reads, so that any wait for a read would be one for all of them; a buffer load counts among the vector memory loads alone.
#pragma once
#include <hip/hip_runtime.h>

namespace hmi {

typedef __attribute__((address_space(3))) void* lds_ptr_t;

#ifdef __HIP_DEVICE_COMPILE__
typedef __amdgpu_buffer_rsrc_t buffer_t;
// Everything from p (uniform) on, raw byte offsets of up to 4 GB.
__device__ __forceinline__ buffer_t buffer_at(const char* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0, 0xFFFFFFFF, 0x00027000);
}
// 16 bytes for each lane, from buffer + lane_off + off + OFF to to + OFF + 16 * lane; to and off uniform.
template <int OFF>
__device__ __forceinline__ void copy_to_lds(buffer_t from, lds_ptr_t to, unsigned lane_off, int off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, to, 16, lane_off, off, OFF, 0);
}
#else   // (the host pass has no such type)
typedef const char* buffer_t;
__device__ buffer_t buffer_at(const char* p);
template <int OFF>
__device__ void copy_to_lds(buffer_t from, lds_ptr_t to, unsigned lane_off, int off);
#endif

}  // namespace hmi
