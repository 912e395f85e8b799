// Device-scope accesses: past the caches that are not coherent between the dies.  What one workgroup writes and another one of
// the same launch reads goes through these.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "frag.h"

namespace mtmc {
namespace device_scope {

using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr int kDeviceScope = 16;  // sc1
constexpr int kReach = 0x40000000;  // bytes that a descriptor covers
__device__ __forceinline__ Rsrc rsrc_of(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kReach, 0x00027000);
}
__device__ __forceinline__ v4u ld16(Rsrc r, int lane_off, int off) {
  return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, kDeviceScope));
}
__device__ __forceinline__ v4f ld16f(Rsrc r, int lane_off, int off) { return __builtin_bit_cast(v4f, ld16(r, lane_off, off)); }
__device__ __forceinline__ void st16(Rsrc r, int lane_off, int off, v4u v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, lane_off, off, kDeviceScope);
}
__device__ __forceinline__ float ld4(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st4(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint2 ld8(const void* p) {
  const uint64_t v = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}
__device__ __forceinline__ void st8(void* p, uint2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), (uint64_t)v.y << 32 | v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A word of memory that workgroups of one launch share.
struct Word {
  uint32_t* p;
  __device__ uint32_t load() const { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ void store(uint32_t v) const { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ uint32_t add(uint32_t v) const { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ uint32_t either(uint32_t v) const { return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ bool swap(uint32_t& seen, uint32_t v) const {
    return __hip_atomic_compare_exchange_strong(p, &seen, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

}  // namespace device_scope
}  // namespace mtmc
