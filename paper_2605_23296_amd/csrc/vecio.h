// 8-element vector load/store helpers for fp32 and bf16 storage, fp32 math.
#pragma once
#include "common.h"

__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
    float4 a = *reinterpret_cast<const float4*>(p);
    float4 b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16* p, float (&v)[8]) {
    bf16x8 a = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (float)a[j];
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16* p, const float (&v)[8]) {
    bf16x8 a;
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = (bf16)v[j];
    *reinterpret_cast<bf16x8*>(p) = a;
}
__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
// index of the wavefront in its workgroup, as a scalar
__device__ __forceinline__ int wave_index() {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#else
    return 0;
#endif
}

// Grouped weight streaming: which k-slice of which column group (of which expert tile) a workgroup of a flat grid takes.  The
// slices of a group are eight workgroups apart, so that they run on one XCD at about the same time (workgroups are dealt to the
// eight XCDs in turn): workgroup 8 (ks a + slice) + x takes group 8a + x.  `tile` may lie past the last one.
struct SliceItem {
    int slice, col, tile;
};
__device__ __forceinline__ SliceItem slice_item(unsigned wg, unsigned ks, unsigned n_cols) {
    const unsigned i = wg >> 3, g = i / ks * 8 + (wg & 7);
    return SliceItem{(int)(i % ks), (int)(g % n_cols), (int)(g / n_cols)};
}
inline int64_t slice_items(int ks, int n_cols, int n_tiles) { return ((int64_t)n_cols * n_tiles + 7) / 8 * 8 * ks; }

// The rotation of one pair, shared with the decode epilogue.  The contraction is written out: left to the compiler it
// changes with the code around it, and a row rotated in a prefill would no longer have the bits of the same row rotated
// in a decode step.
__device__ __forceinline__ void rotate(float lo, float hi, float c, float s, float& olo, float& ohi) {
    olo = fmaf(lo, c, -(hi * s));
    ohi = fmaf(hi, c, lo * s);
}
