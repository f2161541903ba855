// A hand-over between the waves of a workgroup without a barrier: each wave counts itself in, in LDS, behind what
// it has stored, and who waits for the count sees everything that the counted waves stored, in LDS or in global memory.
// That takes a release and an acquire at workgroup scope.  The waves of a workgroup share a compute unit and its vector
// cache, which takes their loads and stores in the order they are issued, so the compiler makes an LDS wait of each
// and keeps the order; it would be free to do neither for relaxed ones.
#pragma once
#include <hip/hip_runtime.h>

// By one lane, behind the stores of its wave (ordered among the wave's lanes by the caller).
__device__ __forceinline__ void count_in(int *count) {
    __hip_atomic_fetch_add(count, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Until n waves have counted themselves in.  A wave that waits has done so itself, and none waits before it has.
__device__ __forceinline__ void wait_for_count(const int *count, int n) {
    while (__hip_atomic_load(count, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < n)
        __builtin_amdgcn_s_sleep(1);
}
