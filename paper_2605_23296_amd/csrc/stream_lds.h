// What the kernels that stream weights through LDS share: waits counted by hand.
#pragma once
#include "common.h"

__device__ __forceinline__ float gs_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// Waits until at most N of this wavefront's loads are in flight (they land in order); its LDS operations are waited for too.
template <int N>
__device__ __forceinline__ void gs_wait() {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(N >= 0 && N < 64, "vector-memory counter is 6 bits");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
    __builtin_amdgcn_sched_barrier(0);
#endif
}
__device__ __forceinline__ void gs_lds_done() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    __builtin_amdgcn_sched_barrier(0);
#endif
}
// index of the wavefront in its workgroup, as a scalar
__device__ __forceinline__ int gs_wave() {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#else
    return 0;
#endif
}
