// What the kernels that stream weights through LDS share: waits counted by hand.
#pragma once
#include "common.h"

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
