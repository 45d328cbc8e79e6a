// span.h -- buffer accesses to one contiguous span of memory (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hicr {

// Global address space (1): plain global_load/global_store instead of flat.
#define GLOBAL __attribute__((address_space(1)))

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// A buffer resource over [base, base + bytes): accesses at or past `bytes`
// read zero and write nothing (the hardware's range check), which lets a
// copy loop run whole rounds without clamping its last one.  base and bytes
// are the same in every lane; base may have any alignment (gfx950 runs the
// HSA unaligned-access mode).
__device__ __forceinline__ rsrc_t span_rsrc(uint64_t base, uint32_t bytes) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)hi << 32) | lo), (short)0,
                                           (int)__builtin_amdgcn_readfirstlane(bytes),
                                           0x00020000);
}

// Accesses with a cache policy (gfx950 bits: 1 = sc0, 2 = nt, 16 = sc1).
template <int Policy>
__device__ __forceinline__ v4i bload(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ void bstore(rsrc_t r, uint32_t off, v4i v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ uint32_t bload8(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, Policy);
}
template <int Policy>
__device__ __forceinline__ void bstore8(rsrc_t r, uint32_t off, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b8((unsigned char)v, r, off, 0, Policy);
}

}  // namespace hicr
