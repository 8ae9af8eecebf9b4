// spin_lds.h -- LDS accesses by 32-bit byte address (a pointer's value in the
// LDS address space), so that address arithmetic stays in one 32-bit register
// and no base of a shared array is added per access.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spin {

typedef uint32_t lds_u2 __attribute__((ext_vector_type(2)));

// Address of an object in LDS.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
__device__ __forceinline__ uint32_t lds_load32(uint32_t at) {
  return *(__attribute__((address_space(3))) const uint32_t*)(uintptr_t)at;
}
__device__ __forceinline__ uint2 lds_load64(uint32_t at) {
  const lds_u2 v = *(__attribute__((address_space(3))) const lds_u2*)(uintptr_t)at;
  return make_uint2(v.x, v.y);
}
__device__ __forceinline__ uint32_t lds_load8(uint32_t at) {
  return *(__attribute__((address_space(3))) const uint8_t*)(uintptr_t)at;
}
__device__ __forceinline__ void lds_store32(uint32_t at, uint32_t v) {
  *(__attribute__((address_space(3))) uint32_t*)(uintptr_t)at = v;
}
__device__ __forceinline__ void lds_store64(uint32_t at, uint2 v) {
  const lds_u2 w = {v.x, v.y};
  *(__attribute__((address_space(3))) lds_u2*)(uintptr_t)at = w;
}

__device__ __forceinline__ float4 lds_load128(uint32_t at) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 v = *(__attribute__((address_space(3))) const f4*)(uintptr_t)at;
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void lds_store128(uint32_t at, const float4& v) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 w = {v.x, v.y, v.z, v.w};
  *(__attribute__((address_space(3))) f4*)(uintptr_t)at = w;
}

}  // namespace spin
