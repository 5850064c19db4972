// Workgroup barriers that leave loads and stores outstanding.
#pragma once

#include <hip/hip_runtime.h>

namespace {

// waits for nothing but what the caller says
__device__ __forceinline__ void bare_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
