// One query row against the keys of one KV head, fp32: shared by the kernels of the fp32 storage mode.
#pragma once
#include "common.h"
#include "vecio.h"

#define F32_KEYS 64

// Sum and maximum over the 16 lanes of a row (every lane receives it), by data movement inside the vector ALU.
template <int CTRL>
__device__ __forceinline__ float row_move(float v) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
#else
    return v;
#endif
}
#define ROW_ROR(n) (0x120 + (n))
__device__ __forceinline__ float row_sum(float v) {
    v += row_move<ROW_ROR(8)>(v);
    v += row_move<ROW_ROR(4)>(v);
    v += row_move<ROW_ROR(2)>(v);
    return v + row_move<ROW_ROR(1)>(v);
}
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, row_move<ROW_ROR(8)>(v));
    v = fmaxf(v, row_move<ROW_ROR(4)>(v));
    v = fmaxf(v, row_move<ROW_ROR(2)>(v));
    return fmaxf(v, row_move<ROW_ROR(1)>(v));
}

// Running softmax state of one query row held across a wavefront: acc[u] is output element state_element(u) of the lane.
struct RowState {
    float m, l, acc[2];
};
__device__ __forceinline__ int state_element(int u) {
    const int lane = threadIdx.x & (WAVE - 1);
    return u * 64 + (lane & 15) * 4 + (lane >> 4);
}

// Sums over the 16 lanes of a row, of 16 values: lane i of the row receives that of v[i].  Every stage adds the half of the
// values that the lane keeps to its partner's (mirrored row, mirrored half row, mirrored and swapped quad): 15 additions
// instead of 64.
// Where only lanes 0 .. N - 1 have something to add (N 8 or 4), the stages beyond N values add zeros to one lane's value: lane i
// takes the N values from fold_value(i) on of lane fold_lane(i) instead, and the stages that are left give the same sum.
template <int CTRL, int H>
__device__ __forceinline__ void fold_stage(float* v, bool upper) {
#pragma unroll
    for (int s = 0; s < H; ++s) {
        const float keep = upper ? v[s + H] : v[s], give = upper ? v[s] : v[s + H];
        v[s] = keep + row_move<CTRL>(give);
    }
}
template <int N>
__device__ __forceinline__ float row_sums(float (&v)[N]) {
    const int i = threadIdx.x & 15;
    if constexpr (N == 16) fold_stage<0x140, 8>(v, (i & 8) != 0);   // row_mirror: lane 15 - i
    if constexpr (N >= 8) fold_stage<0x141, 4>(v, (i & 4) != 0);    // row_half_mirror: 7 - i of the half row
    fold_stage<0x1b, 2>(v, (i & 2) != 0);                           // quad_perm 3 2 1 0
    fold_stage<0xb1, 1>(v, (i & 1) != 0);                           // quad_perm 1 0 3 2
    return v[0];
}
template <int N>
__device__ __forceinline__ int fold_value(int i) {
    return i & ~(N - 1);
}
template <int N>
__device__ __forceinline__ int fold_lane(int i) {
    if (N <= 8 && (i & 8)) i = 15 - i;
    if (N <= 4 && (i & 4)) i = 7 - i;
    return i;
}

// Keys j0 .. j0 + n - 1 (n <= KEYS) of one KV head; qs: the query row (LDS), ps: 64 floats of the wavefront (LDS).
// Both slabs are read 16 lanes to a contiguous run (a key's 64 elements, an output element's 64 keys), four runs per load
// instruction, and the 16 partial sums are added inside the row of lanes; all loads of the piece go out first.  With one
// key, then one output element, per lane every load touched 64 lines: 5.5 us for a decode step over 144 rows.
// KEYS < 64: fewer loads of keys, and an output element's KEYS keys take KEYS / 4 lanes; the sums are the same.
template <int HD, int KEYS>
__device__ __forceinline__ void visit_piece(RowState& st, const float* qs, float* ps, const float* kslab, const float* vslab,
                                            int64_t vstride, int j0, int n, float scale) {
    constexpr int U = HD / 64, S = KEYS / 4;
    const int lane = threadIdx.x & (WAVE - 1), i = lane & 15, g = lane >> 4;
    const int vi = fold_lane<S>(i), vs = fold_value<S>(i);   // keys 4 vi .. of output elements 4 (s + vs) + g
    float4 kv[U][S], vv[U][S];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u)
            kv[u][s] = *reinterpret_cast<const float4*>(kslab + (size_t)(j0 + min(4 * s + g, n - 1)) * HD + u * 64 + i * 4);
    const int key4 = min(4 * vi, (n - 1) & ~3);   // (slab rows are whole 16-byte pieces, j0 is a multiple of 64)
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int u = 0; u < U; ++u)
            vv[u][s] = *reinterpret_cast<const float4*>(vslab + (int64_t)(u * 64 + 4 * (s + vs) + g) * vstride + j0 + key4);
    float4 q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q[u] = *reinterpret_cast<const float4*>(qs + u * 64 + i * 4);
    float dots[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        float a = 0.f;
        if (s < S) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                a = fmaf(q[u].w, kv[u][s].w, fmaf(q[u].z, kv[u][s].z, fmaf(q[u].y, kv[u][s].y, fmaf(q[u].x, kv[u][s].x, a))));
        }
        dots[s] = a;
    }
    const int key = 4 * i + g;   // the key whose probability this lane forms
    const float dot = row_sums(dots);
    const float sc = key < n ? dot * scale : -INFINITY;
    float mx = row_max(sc);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    const float mn = fmaxf(st.m, fmaxf(mx, __shfl_xor(mx, 32, 64)));
    const float corr = expf(st.m - mn);   // exp(-inf) = 0 on the first keys
    const float p = expf(sc - mn);
    float l = row_sum(p);
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    st.l = fmaf(st.l, corr, l);
    st.m = mn;
    ps[key] = p;
    __builtin_amdgcn_wave_barrier();
    const float4 w = *reinterpret_cast<const float4*>(ps + 4 * vi);
    float sums[S];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int s = 0; s < S; ++s) {
            float4 v = vv[u][s];
            if (KEYS < F32_KEYS || n < F32_KEYS) {   // (what lies behind the last key may be anything)
                v.x = 4 * vi < n ? v.x : 0.f;
                v.y = 4 * vi + 1 < n ? v.y : 0.f;
                v.z = 4 * vi + 2 < n ? v.z : 0.f;
                v.w = 4 * vi + 3 < n ? v.w : 0.f;
            }
            sums[s] = fmaf(w.w, v.w, fmaf(w.z, v.z, fmaf(w.y, v.y, w.x * v.x)));
        }
        st.acc[u] = fmaf(st.acc[u], corr, row_sums(sums));
    }
    __builtin_amdgcn_wave_barrier();
}
// n <= MOST keys.  FORMS: by the smallest of the forms that hold them
template <int HD, bool FORMS = false, int MOST = F32_KEYS>
__device__ __forceinline__ void visit_keys(RowState& st, const float* qs, float* ps, const float* kslab, const float* vslab,
                                           int64_t vstride, int j0, int n, float scale) {
    if (FORMS && n <= 16)
        visit_piece<HD, 16>(st, qs, ps, kslab, vslab, vstride, j0, n, scale);
    else if (FORMS && (MOST == 32 || n <= 32))
        visit_piece<HD, 32>(st, qs, ps, kslab, vslab, vstride, j0, n, scale);
    else
        visit_piece<HD, MOST>(st, qs, ps, kslab, vslab, vstride, j0, n, scale);
}

// Output elements state_element(0 ..) of one query row from the states of the four wavefronts that shared its keys, added
// in wavefront order
template <int HD>
__device__ __forceinline__ void merge_states(const float* sm, const float* sl, const float (*sacc)[HD], float (&out)[2]) {
    const int lane = threadIdx.x & (WAVE - 1);
    float m = -INFINITY;
    for (int i = 0; i < 4; ++i) m = fmaxf(m, sm[i]);
    float l = 0.f, a[2] = {0.f, 0.f};
    for (int i = 0; i < 4; ++i) {
        const float f = sl[i] > 0.f ? expf(sm[i] - m) : 0.f;  // a wavefront may have seen no key
        l = fmaf(sl[i], f, l);
#pragma unroll
        for (int u = 0; u < HD / 64; ++u) a[u] = fmaf(sacc[i][u * 64 + lane], f, a[u]);
    }
#pragma unroll
    for (int u = 0; u < HD / 64; ++u) out[u] = a[u] / l;
}
