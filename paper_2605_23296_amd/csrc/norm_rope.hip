// RMSNorm, rotary embedding + KV-cache write, and the row epilogues of the
// decode step.  All of these are bandwidth-bound row kernels: 16-byte loads,
// fp32 arithmetic, one workgroup per row (or per 64-token tile).
#include <algorithm>

#include "common.h"
#include "vecio.h"

#define NT 256

// sum over the workgroup; every thread gets the result
__device__ __forceinline__ float block_sum(float v, float* red) {
    v = wave_sum(v);
    const int w = threadIdx.x / WAVE;
    __syncthreads();
    if ((threadIdx.x & (WAVE - 1)) == 0) red[w] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < NT / WAVE; ++i) t += red[i];
    return t;
}

// ---------------------------------------------------------------------------
// y = x / sqrt(mean(x^2) + eps) * g
// ---------------------------------------------------------------------------
template <typename TI, typename T>
__global__ __launch_bounds__(NT) void rmsnorm_kernel(const TI* __restrict__ x, const T* __restrict__ g,
                                                     T* __restrict__ y, int d, float eps) {
    __shared__ float red[NT / WAVE];
    const TI* xr = x + (size_t)blockIdx.x * d;
    T* yr = y + (size_t)blockIdx.x * d;
    float ss = 0.f;
    for (int c = threadIdx.x * 8; c < d; c += NT * 8) {
        float v[8];
        load8(xr + c, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) ss += v[j] * v[j];
    }
    ss = block_sum(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    for (int c = threadIdx.x * 8; c < d; c += NT * 8) {
        float v[8], gv[8];
        load8(xr + c, v);
        load8(g + c, gv);
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = v[j] * inv * gv[j];
        store8(yr + c, v);
    }
}

int launch_rmsnorm(compact_ctx* ctx, const void* x, bool x_is_f32, const void* g, void* y, int64_t rows, hipStream_t s) {
    if (rows == 0) return COMPACT_OK;
    const int d = ctx->cfg.d_model;
    const dim3 grid((unsigned)rows);
    if (ctx->cfg.dtype == COMPACT_BF16 && x_is_f32)
        rmsnorm_kernel<float, bf16><<<grid, NT, 0, s>>>((const float*)x, (const bf16*)g, (bf16*)y, d, ctx->cfg.rms_eps);
    else if (ctx->cfg.dtype == COMPACT_BF16)
        rmsnorm_kernel<bf16, bf16><<<grid, NT, 0, s>>>((const bf16*)x, (const bf16*)g, (bf16*)y, d, ctx->cfg.rms_eps);
    else
        rmsnorm_kernel<float, float><<<grid, NT, 0, s>>>((const float*)x, (const float*)g, (float*)y, d, ctx->cfg.rms_eps);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Rotary embedding of q and k for a 64-token tile of one block, K rows to the
// K slab, V rows transposed to the V slab.  The rotation angle is formed in
// fp64 (position * theta^(-2i/hd)) so that positions in the thousands do not
// cost fp32 angle precision; cos/sin are then used as fp32.
// A tile's heads are dealt to gridDim.y workgroups (each forms the angles again):
// one workgroup alone walks 20000 pieces of a tile of the 8B-shaped layer in 80
// dependent trips, 75 us whatever the number of tiles; with few tiles that was the
// whole launch (32 tiles: 77 -> 17 us).  Bound with many tiles: HBM (read + write
// of the rows, 8 x 4096: 4.6 TB/s).
// ---------------------------------------------------------------------------
#define ROPE_BATCH 4   // pieces a thread loads before it stores any
template <typename T>
__global__ __launch_bounds__(NT) void rope_kvwrite_kernel(const BlockMeta* __restrict__ meta,
                                                          const TileItem* __restrict__ tiles, T* __restrict__ qkv,
                                                          T* __restrict__ kbase, T* __restrict__ vbase, int Hq, int Hkv,
                                                          int hd, double log2_theta) {
    extern __shared__ char smem[];
    const int half = hd / 2;
    float2* cs = reinterpret_cast<float2*>(smem);                       // [ROPE_TILE][half]
    T* vt = reinterpret_cast<T*>(smem + (size_t)ROPE_TILE * half * 8);  // [ROPE_TILE][hd + 8]
    const int vld = hd + 8;

    const TileItem it = tiles[blockIdx.x];
    const BlockMeta bm = meta[it.block];
    const int p0 = it.row0;
    const int ntok = min(ROPE_TILE, bm.len - p0);
    const int ld = (Hq + 2 * Hkv) * hd;
    T* rows = qkv + (size_t)(bm.row0 + p0) * ld;
    const int part = blockIdx.y, parts = gridDim.y;

    {   // NT is a multiple of half: a thread's frequency is fixed
        const int i = threadIdx.x % half;
        const double inv_freq = exp2(-2.0 * (double)i / (double)hd * log2_theta);
        for (int idx = threadIdx.x; idx < ntok * half; idx += NT) {
            const double ang = (double)(bm.pos_offset + bm.prior + p0 + idx / half) * inv_freq;
            double sn, cn;
            sincos(ang, &sn, &cn);
            cs[idx] = make_float2((float)cn, (float)sn);
        }
    }
    __syncthreads();

    // q heads (in place) and k heads (to the slab): this workgroup's share of the Hq + Hkv heads
    const int chunks = half / 8;
    const int h_lo = part * (Hq + Hkv) / parts, h_hi = (part + 1) * (Hq + Hkv) / parts;
    const int per_tok = (h_hi - h_lo) * chunks, total = ntok * per_tok;
    T* kslab = kbase + bm.slab;
    for (int idx0 = threadIdx.x; idx0 < total; idx0 += NT * ROPE_BATCH) {
        float lo[ROPE_BATCH][8], hi[ROPE_BATCH][8];
#pragma unroll
        for (int u = 0; u < ROPE_BATCH; ++u) {
            const int idx = min(idx0 + u * NT, total - 1);
            const int tok = idx / per_tok, r = idx - tok * per_tok;
            const T* src = rows + (size_t)tok * ld + (h_lo + r / chunks) * hd + (r % chunks) * 8;
            load8(src, lo[u]);
            load8(src + half, hi[u]);
        }
#pragma unroll
        for (int u = 0; u < ROPE_BATCH; ++u) {
            const int idx = idx0 + u * NT;
            if (idx >= total) break;
            const int tok = idx / per_tok, r = idx - tok * per_tok;
            const int head = h_lo + r / chunks, c = r % chunks;
            float olo[8], ohi[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float2 t = cs[tok * half + c * 8 + j];
                rotate(lo[u][j], hi[u][j], t.x, t.y, olo[j], ohi[j]);
            }
            T* dst = rows + (size_t)tok * ld + head * hd + c * 8;
            if (head >= Hq) dst = kslab + ((size_t)(head - Hq) * bm.capacity + bm.prior + p0 + tok) * hd + c * 8;
            store8(dst, olo);
            store8(dst + half, ohi);
        }
    }

    // v heads: stage [tok][hd] in LDS, write [hd][tok]
    T* vslab = vbase + bm.slab;
    for (int kvh = part; kvh < Hkv; kvh += parts) {
        __syncthreads();
        for (int idx = threadIdx.x; idx < ntok * (hd / 8); idx += NT) {
            const int tok = idx / (hd / 8), c = idx - tok * (hd / 8);
            const T* src = rows + (size_t)tok * ld + (Hq + Hkv + kvh) * hd + c * 8;
            float v[8];
            load8(src, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) vt[tok * vld + c * 8 + j] = from_f32<T>(v[j]);
        }
        __syncthreads();
        for (int idx = threadIdx.x; idx < hd * (ROPE_TILE / 8); idx += NT) {
            const int dd = idx / (ROPE_TILE / 8), c = idx - dd * (ROPE_TILE / 8);
            const int t0 = c * 8;
            if (t0 >= ntok) continue;
            T* dst = vslab + ((size_t)kvh * hd + dd) * bm.capacity + bm.prior + p0 + t0;
            if (t0 + 8 <= ntok && (bm.prior & 7) == 0) {   // 16-byte stores need an aligned cache row
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = to_f32(vt[(t0 + j) * vld + dd]);
                store8(dst, v);
            } else {
                for (int j = 0; t0 + j < ntok; ++j) dst[j] = vt[(t0 + j) * vld + dd];
            }
        }
    }
}

int launch_rope_kvwrite(compact_ctx* ctx, const BlockMeta* d_meta, const TileItem* d_tiles, int n_tiles, void* qkv,
                        void* d_k, void* d_v, hipStream_t s) {
    if (n_tiles == 0) return COMPACT_OK;
    const compact_layer_cfg& c = ctx->cfg;
    const double l2t = log2((double)c.rope_theta);
    const size_t es = dtype_size(c.dtype);
    const size_t smem = (size_t)ROPE_TILE * (c.head_dim / 2) * 8 + (size_t)ROPE_TILE * (c.head_dim + 8) * es;
    // about four workgroups per compute unit, no more than one per KV head
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    const int parts = std::max(1, std::min(c.n_kv_heads, (4 * n_cus + n_tiles - 1) / n_tiles));
    const dim3 grid(n_tiles, parts);
    if (c.dtype == COMPACT_BF16)
        rope_kvwrite_kernel<bf16><<<grid, NT, smem, s>>>(d_meta, d_tiles, (bf16*)qkv, (bf16*)d_k, (bf16*)d_v,
                                                         c.n_q_heads, c.n_kv_heads, c.head_dim, l2t);
    else
        rope_kvwrite_kernel<float><<<grid, NT, smem, s>>>(d_meta, d_tiles, (float*)qkv, (float*)d_k, (float*)d_v,
                                                          c.n_q_heads, c.n_kv_heads, c.head_dim, l2t);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Decode row epilogues.  The weight-streaming GEMM leaves ks split-K partials
// [ks][rows][cols] in fp32; these kernels sum them in slice order (all slice
// loads of a thread are issued together) and apply the step that follows.
// ---------------------------------------------------------------------------

// One workgroup (one wavefront) per (head, block token): q heads and k heads are
// rotated at position pos_offset + len + step, q goes to q_out, the K row and
// the V column are appended at cache row len + step.
template <typename T, int KS_UNROLL>
__global__ __launch_bounds__(64) void decode_qkv_epilogue_kernel(const BlockMeta* __restrict__ meta, int n_rows, int step,
                                                                const float* __restrict__ partials, int ks,
                                                                T* __restrict__ q_out, T* __restrict__ kbase,
                                                                T* __restrict__ vbase, int Hq, int Hkv, int hd,
                                                                double log2_theta, const RowNorm norm) {
    const int head = blockIdx.x, b = blockIdx.y;
    const int i = threadIdx.x;
    const int half = hd / 2;
    if (i >= half) return;
    const BlockMeta bm = meta[b];
    const int p = bm.len + step;
    const int ld = (Hq + 2 * Hkv) * hd;
    const size_t ps = (size_t)n_rows * ld;  // stride between split partials
    const float* row = partials + (size_t)b * ld + head * hd;
    float lo = 0.f, hi = 0.f;
    int s = 0;
    for (; s + KS_UNROLL <= ks; s += KS_UNROLL) {
        float a[KS_UNROLL], c[KS_UNROLL];
#pragma unroll
        for (int u = 0; u < KS_UNROLL; ++u) {
            a[u] = row[(s + u) * ps + i];
            c[u] = row[(s + u) * ps + half + i];
        }
#pragma unroll
        for (int u = 0; u < KS_UNROLL; ++u) {
            lo += a[u];
            hi += c[u];
        }
    }
    for (; s < ks; ++s) {
        lo += row[s * ps + i];
        hi += row[s * ps + half + i];
    }
    if (norm.ssq_parts) {
        float ss = 0.f;
        for (int pi = 0; pi < norm.nparts; ++pi) ss += norm.ssq_parts[(size_t)pi * n_rows + b];
        const float rinv = 1.0f / sqrtf(ss * norm.inv_d + norm.eps);
        lo *= rinv;
        hi *= rinv;
    }
    if (head < Hq + Hkv) {
        const double inv_freq = exp2(-2.0 * (double)i / (double)hd * log2_theta);
        double sn, cn;
        sincos((double)(bm.pos_offset + p) * inv_freq, &sn, &cn);
        const float cf = (float)cn, sf = (float)sn;
        float olo, ohi;
        rotate(lo, hi, cf, sf, olo, ohi);
        T* dst = head < Hq ? q_out + ((size_t)b * Hq + head) * hd + i
                           : kbase + bm.slab + ((size_t)(head - Hq) * bm.capacity + p) * hd + i;
        dst[0] = from_f32<T>(olo);
        dst[half] = from_f32<T>(ohi);
    } else {
        T* vcol = vbase + bm.slab + (size_t)(head - Hq - Hkv) * hd * bm.capacity + p;
        vcol[(size_t)i * bm.capacity] = from_f32<T>(lo);
        vcol[(size_t)(i + half) * bm.capacity] = from_f32<T>(hi);
    }
}

int launch_decode_qkv_epilogue(compact_ctx* ctx, const BlockMeta* d_meta, int n_blocks, int step, const float* partials,
                               int ks, void* q_out, void* d_k, void* d_v, hipStream_t s, const RowNorm* norm) {
    const compact_layer_cfg& c = ctx->cfg;
    const RowNorm rn = norm ? *norm : RowNorm{};
    const double l2t = log2((double)c.rope_theta);
    dim3 grid(c.n_q_heads + 2 * c.n_kv_heads, n_blocks);
    if (c.dtype == COMPACT_BF16)
        decode_qkv_epilogue_kernel<bf16, 8><<<grid, 64, 0, s>>>(d_meta, n_blocks, step, partials, ks, (bf16*)q_out,
                                                               (bf16*)d_k, (bf16*)d_v, c.n_q_heads, c.n_kv_heads,
                                                               c.head_dim, l2t, rn);
    else
        decode_qkv_epilogue_kernel<float, 1><<<grid, 64, 0, s>>>(d_meta, n_blocks, step, partials, ks, (float*)q_out,
                                                                (float*)d_k, (float*)d_v, c.n_q_heads, c.n_kv_heads,
                                                                c.head_dim, l2t, rn);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// sum of ks partial float4s at p, p + ps, ... in slice order, loads issued in groups of 8; the last group is of 1, 4 or 8
// (past the end: the last slice again, not added)
template <int U>
__device__ __forceinline__ void add_slices4(const float* __restrict__ p, size_t ps, int n, float4& acc) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const float4*>(p + min(u, n - 1) * ps);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < n) {
            acc.x += v[u].x; acc.y += v[u].y; acc.z += v[u].z; acc.w += v[u].w;
        }
}
__device__ __forceinline__ float4 sum_slices4(const float* __restrict__ p, size_t ps, int ks, float4 acc) {
    int s = 0;
    for (; s + 8 <= ks; s += 8) add_slices4<8>(p + s * ps, ps, 8, acc);
    const int left = ks - s;
    if (left > 4)
        add_slices4<8>(p + s * ps, ps, left, acc);
    else if (left > 1)
        add_slices4<4>(p + s * ps, ps, left, acc);
    else if (left == 1)
        add_slices4<1>(p + s * ps, ps, 1, acc);
    return acc;
}

// ---------------------------------------------------------------------------
// Decode: h = resid + sum_s partial_s (kept in fp32), m = RMSNorm(h; g) in one of the NormRounding forms.
// One workgroup of 1024 threads per row, 4 columns per thread and trip: a row is one or two trips, whose slices are
// requested together; 256 threads for rows of at most 1024 columns (the same sums: the other wavefronts would add zeros).
// Latency-bound: with 256 threads and up to eight trips 10.5 us at 64 rows of 4096, 4 slices; whole steps of 4 to 16 rows of
// d 512 with 1024 threads 41.2 .. 42.4 us, with 256 40.7 .. 41.5.
// ---------------------------------------------------------------------------
#define RN_MAX_D 8192
template <int RN_NT, int RN_TRIPS>
__global__ __launch_bounds__(RN_NT) void residual_norm_kernel(const float* __restrict__ partials, int ks, int rows,
                                                              const bf16* __restrict__ resid, const bf16* __restrict__ g,
                                                              float* __restrict__ h_out, bf16* __restrict__ m_out, int d,
                                                              float eps, NormRounding rounding, float* __restrict__ rinv_out) {
    __shared__ float red[RN_NT / WAVE];
    const int r = blockIdx.x;
    const size_t ps = (size_t)rows * d;
    float4 hv[RN_TRIPS];
    bf16x4 gv[RN_TRIPS];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < RN_TRIPS; ++it) {
        const int c = (it * RN_NT + threadIdx.x) * 4;
        if (c < d) {
            const bf16x4 rv = *reinterpret_cast<const bf16x4*>(resid + (size_t)r * d + c);
            gv[it] = *reinterpret_cast<const bf16x4*>(g + c);
            float4 a = make_float4(to_f32(rv[0]), to_f32(rv[1]), to_f32(rv[2]), to_f32(rv[3]));
            a = sum_slices4(partials + (size_t)r * d + c, ps, ks, a);
            hv[it] = a;
            *reinterpret_cast<float4*>(h_out + (size_t)r * d + c) = a;
            ss += fmaf(a.w, a.w, fmaf(a.z, a.z, fmaf(a.x, a.x, a.y * a.y)));   // (written out: the same in both forms)
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & (WAVE - 1)) == 0) red[threadIdx.x / WAVE] = ss;
    __syncthreads();
    ss = 0.f;
#pragma unroll
    for (int i = 0; i < RN_NT / WAVE; ++i) ss += red[i];
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    const float f = rounding == NORM_LATER ? 1.0f : inv;
    if (rounding == NORM_LATER && threadIdx.x == 0) rinv_out[r] = inv;
#pragma unroll
    for (int it = 0; it < RN_TRIPS; ++it) {
        const int c = (it * RN_NT + threadIdx.x) * 4;
        if (c < d) {
            bf16x4 m;
            m[0] = (bf16)(hv[it].x * f * to_f32(gv[it][0]));
            m[1] = (bf16)(hv[it].y * f * to_f32(gv[it][1]));
            m[2] = (bf16)(hv[it].z * f * to_f32(gv[it][2]));
            m[3] = (bf16)(hv[it].w * f * to_f32(gv[it][3]));
            *reinterpret_cast<bf16x4*>(m_out + (size_t)r * d + c) = m;
        }
    }
}

int launch_residual_norm(compact_ctx* ctx, const float* partials, int ks, const void* resid, const void* g,
                         void* h_out, void* m_out, int rows, hipStream_t s, NormRounding rounding, float* rinv_out) {
    const compact_layer_cfg& c = ctx->cfg;
    if (rounding == NORM_LATER && !rinv_out) return set_err(ctx, COMPACT_EINVAL, "no room for the rows' 1 / rms");
    if (c.d_model > RN_MAX_D) return set_err(ctx, COMPACT_ESHAPE, "d_model above 8192 is not supported by the decode row kernels");
    if (c.d_model <= 1024)
        residual_norm_kernel<256, 1><<<rows, 256, 0, s>>>(partials, ks, rows, (const bf16*)resid, (const bf16*)g, (float*)h_out,
                                                          (bf16*)m_out, c.d_model, c.rms_eps, rounding, rinv_out);
    else
        residual_norm_kernel<1024, RN_MAX_D / 4096><<<rows, 1024, 0, s>>>(partials, ks, rows, (const bf16*)resid, (const bf16*)g,
                                                                         (float*)h_out, (bf16*)m_out, c.d_model, c.rms_eps, rounding,
                                                                         rinv_out);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Decode: act = silu(gate) * up, gate/up = sum of partials of the stacked
// projection [rows, 2F]
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NT) void swiglu_reduce_kernel(const float* __restrict__ partials, int ks, int rows,
                                                           bf16* __restrict__ act, int F) {
    const int r = blockIdx.y;
    const int c = blockIdx.x * NT + threadIdx.x;
    if (c >= F) return;
    const size_t ps = (size_t)rows * 2 * F;
    float gt = 0.f, up = 0.f;
    for (int s = 0; s < ks; ++s) {
        gt += partials[s * ps + (size_t)r * 2 * F + c];
        up += partials[s * ps + (size_t)r * 2 * F + F + c];
    }
    const float sg = gt / (1.0f + expf(-gt));
    act[(size_t)r * F + c] = (bf16)(sg * up);
}

int launch_swiglu_reduce(compact_ctx* ctx, const float* partials, int ks, void* act, int rows, int F, hipStream_t s) {
    dim3 grid((F + NT - 1) / NT, rows);
    swiglu_reduce_kernel<<<grid, NT, 0, s>>>(partials, ks, rows, (bf16*)act, F);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Decode: y = resid (fp32) + sum_s partial_s ; 4 columns per thread
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NT) void residual_reduce_kernel(const float* __restrict__ partials, int ks, int rows,
                                                             const float* __restrict__ resid, bf16* __restrict__ y,
                                                             int cols) {
    const size_t i = ((size_t)blockIdx.x * NT + threadIdx.x) * 4;
    const size_t total = (size_t)rows * cols;
    if (i >= total) return;
    float4 a = *reinterpret_cast<const float4*>(resid + i);
    a = sum_slices4(partials + i, total, ks, a);
    y[i] = (bf16)(a.x);
    y[i + 1] = (bf16)(a.y);
    y[i + 2] = (bf16)(a.z);
    y[i + 3] = (bf16)(a.w);
}

int launch_residual_reduce(compact_ctx* ctx, const float* partials, int ks, const void* resid, void* y, int rows,
                           int cols, hipStream_t s) {
    const size_t total = (size_t)rows * cols;  // cols is a multiple of 64
    const unsigned grid = (unsigned)((total / 4 + NT - 1) / NT);
    residual_reduce_kernel<<<grid, NT, 0, s>>>(partials, ks, rows, (const float*)resid, (bf16*)y, cols);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// y_last[b] = y[last row of block b]
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(NT) void gather_last_rows_kernel(const BlockMeta* __restrict__ meta,
                                                              const T* __restrict__ y, T* __restrict__ y_last, int d) {
    const BlockMeta bm = meta[blockIdx.x];
    const T* src = y + (size_t)(bm.row0 + bm.len - 1) * d;
    T* dst = y_last + (size_t)blockIdx.x * d;
    for (int c = threadIdx.x; c < d; c += NT) dst[c] = src[c];
}

int launch_gather_last_rows(compact_ctx* ctx, const BlockMeta* d_meta, int n_blocks, const void* y, void* y_last,
                            hipStream_t s) {
    if (ctx->cfg.dtype == COMPACT_BF16)
        gather_last_rows_kernel<bf16><<<n_blocks, NT, 0, s>>>(d_meta, (const bf16*)y, (bf16*)y_last, ctx->cfg.d_model);
    else
        gather_last_rows_kernel<float><<<n_blocks, NT, 0, s>>>(d_meta, (const float*)y, (float*)y_last, ctx->cfg.d_model);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Row mover of the mixed-batch scheduler: packed row i is read from / written to
// the row a table names.  Table value v >= 0: row v of base 0; v <= -2: row
// (-v - 2) of base 1; v == -1: no row (skip).  A null table means row i of base 0.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(NT) void move_rows_kernel(const T* __restrict__ src0, const T* __restrict__ src1,
                                                       const int32_t* __restrict__ src_tab, T* __restrict__ dst0,
                                                       T* __restrict__ dst1, const int32_t* __restrict__ dst_tab, int d) {
    const int i = blockIdx.x;
    const int sv = src_tab ? src_tab[i] : i;
    const int dv = dst_tab ? dst_tab[i] : i;
    if (sv == -1 || dv == -1) return;
    const T* src = sv >= 0 ? src0 + (size_t)sv * d : src1 + (size_t)(-sv - 2) * d;
    T* dst = dv >= 0 ? dst0 + (size_t)dv * d : dst1 + (size_t)(-dv - 2) * d;
    for (int c = threadIdx.x; c < d; c += NT) dst[c] = src[c];
}

int launch_move_rows(compact_ctx* ctx, const void* src0, const void* src1, const int32_t* src_tab, void* dst0, void* dst1,
                     const int32_t* dst_tab, int rows, hipStream_t s) {
    if (rows == 0) return COMPACT_OK;
    const int d = ctx->cfg.d_model;
    if (ctx->cfg.dtype == COMPACT_BF16)
        move_rows_kernel<bf16><<<rows, NT, 0, s>>>((const bf16*)src0, (const bf16*)src1, src_tab, (bf16*)dst0, (bf16*)dst1, dst_tab, d);
    else
        move_rows_kernel<float><<<rows, NT, 0, s>>>((const float*)src0, (const float*)src1, src_tab, (float*)dst0, (float*)dst1, dst_tab, d);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
