// spin_launch.h -- what launch functions share.
#pragma once

#include <hip/hip_runtime.h>

#include <initializer_list>

#include "spin_once.h"

namespace spin {

// Lets workgroups of the kernels have `bytes` of dynamic LDS on the current device: set once for it (`once` belongs to
// this set of kernels).
inline hipError_t allow_lds(OncePerDevice& once, std::initializer_list<const void*> kernels, int bytes) {
  int device = -1;
  (void)hipGetDevice(&device);
  return once.run(device, hipSuccess, [&] {
    for (const void* k : kernels) {
      const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  });
}

}  // namespace spin
