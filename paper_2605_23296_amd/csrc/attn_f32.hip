// fp32 attention of the fp32 storage mode.  A wavefront takes its keys 64 at a
// time (attn_f32.h): scores, one wave-wide maximum and sum, then P V (the V slab is
// transposed).  So the dependent chain is one reduction per 64 keys; visiting one key
// at a time it was 14.6 us for a decode step over 144 rows and 65 us for the prefill
// of four blocks of 128.
#include "attn_f32.h"

// head_dim 128: few keys take the forms for 16 and 32, and a call whose rows all have at most MOST = 32 a kernel of these alone.
// The form for 64 keeps the 64 loads of a piece in 256 registers, so one wavefront per SIMD; calls of short blocks, 8 heads,
// lost by it against lane = key with 90 registers (64 blocks of 40 tokens 364 -> 381 us, 300 of 5 225 -> 264; now 340 and 205).
// At head_dim 64 (163 registers) the one form is the faster one throughout, and so it is in a decode step.
template <int HD, int MOST>
__global__ __launch_bounds__(256) void attn_prefill_f32_kernel(const BlockMeta* __restrict__ meta,
                                                               const float* __restrict__ qkv,
                                                               const float* __restrict__ kbase,
                                                               const float* __restrict__ vbase, float* __restrict__ o,
                                                               int Hq, int Hkv, float scale) {
    __shared__ __attribute__((aligned(16))) float qs[4][HD], ps[4][F32_KEYS];
    const BlockMeta bm = meta[blockIdx.z];
    const int w = threadIdx.x / WAVE;
    const int i = blockIdx.x * 4 + w;
    if (i >= bm.len) return;   // (no workgroup barrier below)
    const int h = blockIdx.y, kvh = h / (Hq / Hkv);
    const int lane = threadIdx.x & (WAVE - 1);
    const int ld = (Hq + 2 * Hkv) * HD;
    const float* qrow = qkv + (size_t)(bm.row0 + i) * ld + h * HD;
#pragma unroll
    for (int u = 0; u < HD / 64; ++u) qs[w][u * 64 + lane] = qrow[u * 64 + lane];
    __builtin_amdgcn_wave_barrier();
    const float* kslab = kbase + bm.slab + (size_t)kvh * bm.capacity * HD;
    const float* vslab = vbase + bm.slab + (size_t)kvh * HD * bm.capacity;
    RowState st = {-INFINITY, 0.f, {0.f, 0.f}};
    const int n_keys = bm.prior + i + 1;
    for (int j = 0; j < n_keys; j += F32_KEYS)
        visit_keys<HD, HD == 128, MOST>(st, qs[w], ps[w], kslab, vslab, bm.capacity, j, min(F32_KEYS, n_keys - j), scale);
    float* orow = o + (size_t)(bm.row0 + i) * Hq * HD + h * HD;
#pragma unroll
    for (int u = 0; u < HD / 64; ++u) orow[state_element(u)] = st.acc[u] / st.l;
}

int launch_attn_prefill_f32(compact_ctx* ctx, const BlockMeta* d_meta, int n_blocks, int max_len, int max_keys, const float* qkv,
                            const float* d_k, const float* d_v, float* o, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    dim3 grid((max_len + 3) / 4, c.n_q_heads, n_blocks);
    const float scale = 1.0f / sqrtf((float)c.head_dim);
    if (c.head_dim == 128 && max_keys <= 32)
        attn_prefill_f32_kernel<128, 32><<<grid, 256, 0, s>>>(d_meta, qkv, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, scale);
    else if (c.head_dim == 128)
        attn_prefill_f32_kernel<128, F32_KEYS><<<grid, 256, 0, s>>>(d_meta, qkv, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, scale);
    else
        attn_prefill_f32_kernel<64, F32_KEYS><<<grid, 256, 0, s>>>(d_meta, qkv, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, scale);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// one workgroup per (head, block); its 4 wavefronts take the 64-key pieces w, w+4, ... and
// their states are merged in wavefront order
template <int HD>
__global__ __launch_bounds__(256) void attn_decode_f32_kernel(const BlockMeta* __restrict__ meta, int step,
                                                              const float* __restrict__ q,
                                                              const float* __restrict__ kbase,
                                                              const float* __restrict__ vbase, float* __restrict__ o,
                                                              int Hq, int Hkv, float scale) {
    __shared__ __attribute__((aligned(16))) float qs[HD], ps[4][F32_KEYS];
    __shared__ float sm[4], sl[4], sacc[4][HD];
    const BlockMeta bm = meta[blockIdx.y];
    const int n_keys = bm.len + step + 1;  // the appended row is included
    const int h = blockIdx.x, kvh = h / (Hq / Hkv);
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    if (threadIdx.x < HD) qs[threadIdx.x] = q[(size_t)blockIdx.y * Hq * HD + h * HD + threadIdx.x];
    __syncthreads();
    const float* kslab = kbase + bm.slab + (size_t)kvh * bm.capacity * HD;
    const float* vslab = vbase + bm.slab + (size_t)kvh * HD * bm.capacity;
    RowState st = {-INFINITY, 0.f, {0.f, 0.f}};
    for (int j = w * F32_KEYS; j < n_keys; j += 4 * F32_KEYS)
        visit_keys<HD>(st, qs, ps[w], kslab, vslab, bm.capacity, j, min(F32_KEYS, n_keys - j), scale);
    if (lane == 0) {
        sm[w] = st.m;
        sl[w] = st.l;
    }
#pragma unroll
    for (int u = 0; u < HD / 64; ++u) sacc[w][u * 64 + lane] = st.acc[u];
    __syncthreads();
    if (w == 0) {
        float out[2];
        merge_states<HD>(sm, sl, sacc, out);
        float* orow = o + (size_t)blockIdx.y * Hq * HD + h * HD;
#pragma unroll
        for (int u = 0; u < HD / 64; ++u) orow[state_element(u)] = out[u];
    }
}

int launch_attn_decode_f32(compact_ctx* ctx, const BlockMeta* d_meta, int n_blocks, int step, const float* q,
                           const float* d_k, const float* d_v, float* o, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    dim3 grid(c.n_q_heads, n_blocks);
    const float scale = 1.0f / sqrtf((float)c.head_dim);
    if (c.head_dim == 128)
        attn_decode_f32_kernel<128><<<grid, 256, 0, s>>>(d_meta, step, q, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, scale);
    else
        attn_decode_f32_kernel<64><<<grid, 256, 0, s>>>(d_meta, step, q, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, scale);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
