// Raw buffer access: an offset at or beyond the buffer's size reads 0 and drops
// a store, which replaces the per-lane bounds tests of loads and stores.
#pragma once

#include <hip/hip_runtime.h>

namespace c0ip {
namespace rawbuf {

constexpr unsigned kOff = 0x80000000u;  // an offset outside every buffer
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
// scalar: a wave-uniform offset added to off
template <typename T>
__device__ __forceinline__ T load(__amdgpu_buffer_rsrc_t r, unsigned off, int scalar = 0) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, scalar, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, scalar, 0));
}
template <typename T>
__device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, unsigned off, T v) {
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off, 0, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off, 0, 0);
}

}  // namespace rawbuf
}  // namespace c0ip
