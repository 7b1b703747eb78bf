// Mixture-of-experts plumbing: top-k routing from fp32 logits, the
// token -> expert permutation (histogram, scan, scatter, row-tile map for the
// grouped GEMM) and the weighted un-permute + residual.
#include "common.h"
#include "vecio.h"

// ---------------------------------------------------------------------------
// top-k of E fp32 logits per row (descending, equal logits -> lower index),
// gate = softmax over the selected logits.  One wavefront per row; lane l owns
// experts l, l+64, l+128, l+192.
// ---------------------------------------------------------------------------
// (nothing is indexed by a loop variable that is not unrolled away: that would put the values into scratch memory)
__device__ __forceinline__ void topk_row(float (&v)[4], int lane, int k, int32_t* idx, float* gate) {
    float sel_v = 0.f, top = 0.f;   // lane j: the j-th selected logit and its expert
    int sel_i = 0;
    for (int j = 0; j < k; ++j) {
        // lane-local best (lower index wins ties: scan in increasing index order with strict >)
        float bv = v[0];
        int bi = lane;
#pragma unroll
        for (int i = 1; i < 4; ++i)
            if (v[i] > bv) {
                bv = v[i];
                bi = lane + i * 64;
            }
        // wavefront arg-max on (value desc, index asc)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (ov > bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        if (j == 0) top = bv;
        if (lane == j) {
            sel_v = bv;
            sel_i = bi;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (bi == lane + i * 64) v[i] = -INFINITY;   // remove the winner
    }
    top = __shfl(top, 0, 64);
    const float p = lane < k ? expf(sel_v - top) : 0.f;
    float den = 0.f;
    for (int j = 0; j < k; ++j) den += __shfl(p, j, 64);
    if (lane < k) {
        idx[lane] = sel_i;
        gate[lane] = p / den;
    }
}
// the row's logits from ks split-K partials [ks][rows][E]: all partials of the lane's experts are requested before the
// first is used (slices in groups of 8), then added in slice order
__device__ __forceinline__ void sum_logits(const float* __restrict__ partials, int ks, int64_t rows, int64_t row, int E, int lane,
                                           float (&v)[4]) {
    float a[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < ks; s0 += 8) {
        float pv[4][8];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = lane + i * 64;
                pv[i][u] = (e < E && s0 + u < ks) ? partials[((size_t)(s0 + u) * rows + row) * E + e] : 0.f;
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < ks) a[i] += pv[i][u];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = lane + i * 64 < E ? a[i] : -INFINITY;
}
// ks > 0: the logits arrive as ks split-K partials [ks][rows][E]; they are summed in
// slice order here and the sums are written to `logits`.
__global__ __launch_bounds__(256) void topk_route_kernel(float* __restrict__ logits, const float* __restrict__ partials, int ks,
                                                         int64_t rows, int E, int k, int32_t* __restrict__ idx,
                                                         float* __restrict__ gate) {
    const int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
    if (row >= rows) return;
    const int lane = threadIdx.x & (WAVE - 1);
    float v[4];
    if (ks > 0) {
        sum_logits(partials, ks, rows, row, E, lane, v);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (lane + i * 64 < E) logits[row * E + lane + i * 64] = v[i];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = lane + i * 64;
            v[i] = e < E ? logits[row * E + e] : -INFINITY;
        }
    }
    topk_row(v, lane, k, idx + row * k, gate + row * k);
}

int launch_moe_route(compact_ctx* ctx, const void* m, const void* w_router, int64_t rows, int32_t* idx, float* gate,
                     float* logits, hipStream_t s, float* partials_ws) {
    if (rows == 0) return COMPACT_OK;
    const compact_layer_cfg& c = ctx->cfg;
    int rc;
    if (c.dtype == COMPACT_BF16 && partials_ws && rows <= 64 && c.n_experts % 16 == 0 && c.d_model % 64 == 0) {
        // a few decode rows: the router matrix is streamed once by the weight-streaming kernel
        const int ks = skinny_ksplit((int)rows, c.n_experts, c.d_model);
        rc = launch_gemm_skinny(ctx, (const bf16*)m, (const bf16*)w_router, partials_ws, (int)rows, c.n_experts, c.d_model, ks, s);
        if (rc != COMPACT_OK) return rc;
        topk_route_kernel<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(logits, partials_ws, ks, rows, c.n_experts, c.top_k, idx, gate);
        LAUNCH_CHECK(ctx);
        return COMPACT_OK;
    }
    if (c.dtype == COMPACT_BF16)
        rc = launch_gemm_bf16(ctx, (const bf16*)m, (const bf16*)w_router, nullptr, false, (bf16*)logits, rows,
                              c.n_experts, c.d_model, 2, nullptr, s);
    else
        rc = launch_gemm_f32(ctx, (const float*)m, (const float*)w_router, nullptr, logits, rows, c.n_experts,
                             c.d_model, 0, nullptr, s);
    if (rc != COMPACT_OK) return rc;
    topk_route_kernel<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(logits, nullptr, 0, rows, c.n_experts, c.top_k, idx, gate);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// permutation plan
// ---------------------------------------------------------------------------
__global__ void zero_i32_kernel(int32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// rank[i] = position of entry i among the entries routed to the same expert
// (any order: the order of rows inside an expert's group does not enter the
// arithmetic).  Workgroup-local ranks from an LDS histogram, one global
// reservation per (workgroup, expert).
__global__ __launch_bounds__(256) void expert_rank_kernel(const int32_t* __restrict__ idx, int64_t n, int E,
                                                          int32_t* __restrict__ counts, int32_t* __restrict__ rank) {
    __shared__ int32_t lc[256], base[256];
    const int t = threadIdx.x;
    lc[t] = 0;
    __syncthreads();
    constexpr int PER = 4;
    int e[PER], lr[PER];
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + t) * PER;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        e[j] = -1;
        if (i0 + j < n) {
            e[j] = idx[i0 + j];
            lr[j] = atomicAdd(&lc[e[j]], 1);
        }
    }
    __syncthreads();
    if (t < E && lc[t] > 0) base[t] = atomicAdd(&counts[t], lc[t]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (e[j] >= 0) rank[i0 + j] = base[e[j]] + lr[j];
}

// offsets = exclusive scan of counts; row-tile map for the grouped GEMM
__global__ __launch_bounds__(256) void expert_scan_kernel(const int32_t* __restrict__ counts, int E, int mtile,
                                                          int32_t* __restrict__ offsets, int32_t* __restrict__ tile_expert,
                                                          int32_t* __restrict__ tile_row0, int32_t* __restrict__ tile_rows,
                                                          int max_mtiles) {
    __shared__ int32_t off[257], toff[257];
    if (threadIdx.x == 0) {
        int a = 0, b = 0;
        for (int e = 0; e < E; ++e) {
            off[e] = a;
            toff[e] = b;
            a += counts[e];
            b += (counts[e] + mtile - 1) / mtile;
        }
        off[E] = a;
        toff[E] = b;
    }
    __syncthreads();
    for (int e = threadIdx.x; e <= E; e += 256) offsets[e] = off[e];
    for (int e = threadIdx.x; e < E; e += 256) {
        const int cnt = off[e + 1] - off[e];
        for (int i = 0; toff[e] + i < toff[e + 1]; ++i) {
            const int ti = toff[e] + i;
            tile_expert[ti] = e;
            tile_row0[ti] = off[e] + i * mtile;
            tile_rows[ti] = min(mtile, cnt - i * mtile);
        }
    }
    for (int ti = toff[E] + threadIdx.x; ti < max_mtiles; ti += 256) {
        tile_expert[ti] = -1;
        tile_row0[ti] = 0;
        tile_rows[ti] = 0;
    }
}

__global__ __launch_bounds__(256) void expert_scatter_kernel(const int32_t* __restrict__ idx, const float* __restrict__ gate,
                                                             const int32_t* rank,
                                                             const int32_t* __restrict__ offsets, int64_t n, int k,
                                                             int32_t* __restrict__ sorted_token,
                                                             float* __restrict__ sorted_gate, int32_t* slot_of) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int pos = offsets[idx[i]] + rank[i];
    sorted_token[pos] = (int32_t)(i / k);
    sorted_gate[pos] = gate[i];
    slot_of[i] = pos;
}

// The whole plan in one workgroup, for at most 256 routed entries (a decode step) and
// at most 256 experts: rank = number of earlier entries with the same expert (so the
// order inside an expert's group is the token order), counts, scan, tile map, scatter.
// Threads 0 .. 255 work (all threads of the workgroup pass the barriers); thread t holds entry t: its expert (-1: none) and gate.
struct PlanOut {
    int32_t *counts, *offsets, *tile_expert, *tile_row0, *tile_rows, *sorted_token, *slot_of;
    float* sorted_gate;
    int max_mtiles;
};
__device__ __forceinline__ void plan_small(int t, int my, float gate, int n, int k, int E, int mtile, const PlanOut& o) {
    __shared__ __attribute__((aligned(16))) int32_t se[256];
    __shared__ int32_t off[257], toff[257], wsum[4][2];
    const bool on = t < 256;
    if (on) se[t] = my;
    __syncthreads();
    int rank = 0, cnt = 0;
    if (on) {
        for (int j = 0; j < n; j += 16) {   // (entries past n hold -1)
            int4 e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = *reinterpret_cast<const int4*>(se + j + 4 * u);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q[4] = {e[u].x, e[u].y, e[u].z, e[u].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    rank += (j + 4 * u + i < t && q[i] == my) ? 1 : 0;
                    cnt += q[i] == t ? 1 : 0;
                }
            }
        }
        if (t < E) o.counts[t] = cnt;
    }
    // exclusive scans of the counts and of the tiles per expert over the 256 threads (thread e = expert e): within each
    // wavefront by shuffles, then the wavefronts' sums
    int a = on && t < E ? cnt : 0, b = (a + mtile - 1) / mtile;
    const int lane = t & 63;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const int x = __shfl_up(a, st, 64), y = __shfl_up(b, st, 64);
        if (lane >= st) {
            a += x;
            b += y;
        }
    }
    if (on && lane == 63) {
        wsum[t >> 6][0] = a;
        wsum[t >> 6][1] = b;
    }
    __syncthreads();
    if (on) {
        for (int w = 0; w < (t >> 6); ++w) {
            a += wsum[w][0];
            b += wsum[w][1];
        }
        off[t + 1] = a;
        toff[t + 1] = b;
        if (t == 0) off[0] = toff[0] = 0;
    }
    __syncthreads();
    if (!on) return;
    for (int e = t; e <= E; e += 256) o.offsets[e] = off[e];
    if (t < E) {
        for (int i = 0; toff[t] + i < toff[t + 1]; ++i) {
            const int ti = toff[t] + i;
            o.tile_expert[ti] = t;
            o.tile_row0[ti] = off[t] + i * mtile;
            o.tile_rows[ti] = min(mtile, cnt - i * mtile);
        }
    }
    for (int ti = toff[E] + t; ti < o.max_mtiles; ti += 256) {
        o.tile_expert[ti] = -1;
        o.tile_row0[ti] = 0;
        o.tile_rows[ti] = 0;
    }
    if (my >= 0) {
        const int pos = off[my] + rank;
        o.sorted_token[pos] = t / k;
        o.sorted_gate[pos] = gate;
        o.slot_of[t] = pos;
    }
}

__global__ __launch_bounds__(256) void moe_plan_small_kernel(const int32_t* __restrict__ idx, const float* __restrict__ gate, int n,
                                                             int k, int E, int mtile, const PlanOut out) {
    const int t = threadIdx.x;
    plan_small(t, t < n ? idx[t] : -1, t < n ? gate[t] : 0.f, n, k, E, mtile, out);
}

// Decode: logits (split-K partials), top-k and plan in one workgroup of 16 wavefronts, a row per wavefront.
// Latency-bound, so the launch between the two is what it saves: 8.0 + 7.0 us apart, 9.7 us together (16 rows, 128
// experts, top-4).  More than 16 rows would take a second trip to memory one after the other, and are faster as two
// launches with a wavefront per row over the whole chip: whole steps of 17 / 32 / 64 rows of the 120B-shaped layer with
// 4-bit experts 224 / 310 / 443 us here, 223 / 307 / 431 apart.
#define ROUTE_PLAN_ROWS 16
__global__ __launch_bounds__(ROUTE_PLAN_ROWS * 64) void route_plan_kernel(const float* __restrict__ partials, int ks, int rows,
                                                                          int E, int k, int32_t* __restrict__ idx,
                                                                          float* __restrict__ gate, int mtile, const PlanOut out) {
    __shared__ int32_t s_idx[ROUTE_PLAN_ROWS * 8];   // (top_k is at most 8)
    __shared__ float s_gate[ROUTE_PLAN_ROWS * 8];
    const int t = threadIdx.x, lane = t & 63;
    const int row = t >> 6;
    if (row < rows) {
        float v[4];
        sum_logits(partials, ks, rows, row, E, lane, v);
        topk_row(v, lane, k, s_idx + row * k, s_gate + row * k);
    }
    __syncthreads();
    const int n = rows * k;
    if (t < n) {
        idx[t] = s_idx[t];
        gate[t] = s_gate[t];
    }
    plan_small(t, t < n ? s_idx[t] : -1, t < n ? s_gate[t] : 0.f, n, k, E, mtile, out);
}

static PlanOut plan_out(const MoePlan& p) {
    return PlanOut{p.counts, p.offsets, p.tile_expert, p.tile_row0, p.tile_rows, p.sorted_token, p.slot_of, p.sorted_gate, p.max_mtiles};
}

bool moe_route_plan_supported(const compact_layer_cfg& c, int rows) {
    return c.dtype == COMPACT_BF16 && rows <= ROUTE_PLAN_ROWS && c.n_experts % 16 == 0 && c.n_experts <= 256 &&
           c.d_model % 64 == 0;
}

int launch_moe_route_plan(compact_ctx* ctx, const bf16* hg, const RowNorm* norm, bf16* m, const bf16* w_router, int rows,
                          int32_t* idx, float* gate, float* partials_ws, int mtile, const MoePlan& plan, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    if (!moe_route_plan_supported(c, rows)) return set_err(ctx, COMPACT_ESHAPE, "one-workgroup routing takes at most 16 rows");
    const int ks = skinny_ksplit(rows, c.n_experts, c.d_model);
    int rc;
    if (norm)
        rc = launch_gemm_skinny_rownorm(ctx, hg, *norm, m, w_router, partials_ws, rows, c.n_experts, c.d_model, ks, s);
    else
        rc = launch_gemm_skinny(ctx, m, w_router, partials_ws, rows, c.n_experts, c.d_model, ks, s);
    if (rc != COMPACT_OK) return rc;
    route_plan_kernel<<<1, ROUTE_PLAN_ROWS * 64, 0, s>>>(partials_ws, ks, rows, c.n_experts, c.top_k, idx, gate, mtile, plan_out(plan));
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

int launch_moe_plan(compact_ctx* ctx, const int32_t* idx, const float* gate, int64_t rows, int mtile,
                    const MoePlan& plan, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    const int64_t n = rows * c.top_k;
    if (n == 0) return COMPACT_OK;
    if (n <= 256 && c.n_experts <= 256) {
        moe_plan_small_kernel<<<1, 256, 0, s>>>(idx, gate, (int)n, c.top_k, c.n_experts, mtile, plan_out(plan));
        LAUNCH_CHECK(ctx);
        return COMPACT_OK;
    }
    zero_i32_kernel<<<1, 256, 0, s>>>(plan.counts, c.n_experts);
    // slot_of doubles as the rank buffer until the scatter overwrites it entry by entry
    expert_rank_kernel<<<(unsigned)((n + 1023) / 1024), 256, 0, s>>>(idx, n, c.n_experts, plan.counts, plan.slot_of);
    expert_scan_kernel<<<1, 256, 0, s>>>(plan.counts, c.n_experts, mtile, plan.offsets, plan.tile_expert, plan.tile_row0,
                                         plan.tile_rows, plan.max_mtiles);
    expert_scatter_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(idx, gate, plan.slot_of, plan.offsets, n, c.top_k,
                                                                      plan.sorted_token, plan.sorted_gate, plan.slot_of);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// y[t] = h[t] + sum_j expert_out[slot_of[t*k + j]]   (rows already gate-scaled)
// ---------------------------------------------------------------------------
template <typename T, typename HT>
__global__ __launch_bounds__(256) void moe_combine_kernel(const T* __restrict__ expert_out, const HT* __restrict__ hres,
                                                          const int32_t* __restrict__ slot_of, int k, int d,
                                                          T* __restrict__ y) {
    const int64_t row = blockIdx.x;
    for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
        float acc[8];
        load8(hres + row * d + c, acc);
        for (int j = 0; j < k; ++j) {
            float v[8];
            load8(expert_out + (int64_t)slot_of[row * k + j] * d + c, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += v[e];
        }
        store8(y + row * d + c, acc);
    }
}

int launch_moe_combine(compact_ctx* ctx, const void* expert_out, const void* h, bool h_is_f32, const int32_t* slot_of,
                       int64_t rows, void* y, hipStream_t s) {
    if (rows == 0) return COMPACT_OK;
    const compact_layer_cfg& c = ctx->cfg;
    const unsigned g = (unsigned)rows;
    if (c.dtype == COMPACT_BF16 && h_is_f32)
        moe_combine_kernel<bf16, float><<<g, 256, 0, s>>>((const bf16*)expert_out, (const float*)h, slot_of, c.top_k, c.d_model, (bf16*)y);
    else if (c.dtype == COMPACT_BF16)
        moe_combine_kernel<bf16, bf16><<<g, 256, 0, s>>>((const bf16*)expert_out, (const bf16*)h, slot_of, c.top_k, c.d_model, (bf16*)y);
    else
        moe_combine_kernel<float, float><<<g, 256, 0, s>>>((const float*)expert_out, (const float*)h, slot_of, c.top_k, c.d_model, (float*)y);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Decode: y[t] = h[t] + sum_j gate_j * (sum_s P[s][slot_of[t*k + j]]), with the
// split-K partials of the routed down projection still in fp32: one rounding.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void moe_combine_partials_kernel(const float* __restrict__ P, int ks, int64_t total_rows,
                                                                   const float* __restrict__ hres,
                                                                   const int32_t* __restrict__ slot_of,
                                                                   const float* __restrict__ sorted_gate, int k, int d,
                                                                   bf16* __restrict__ y) {
    const int64_t row = blockIdx.y;
    const int c = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (c >= d) return;
    // the loads go out in three waves (all slots, then all gate weights, then per expert all its slices, 8 at a
    // time) instead of one after the other; the sums keep their order: slices in slice order, experts in j order
    constexpr int KMAX = 8;   // top_k <= 8
    int64_t slot[KMAX];
    float gw[KMAX];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) slot[j] = slot_of[row * k + min(j, k - 1)];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) gw[j] = sorted_gate[slot[j]];
    float4 acc = *reinterpret_cast<const float4*>(hres + row * d + c);
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        if (j >= k) break;
        float4 e = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int s0 = 0; s0 < ks; s0 += 8) {
            float4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = *reinterpret_cast<const float4*>(P + ((int64_t)min(s0 + u, ks - 1) * total_rows + slot[j]) * d + c);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (s0 + u < ks) { e.x += v[u].x; e.y += v[u].y; e.z += v[u].z; e.w += v[u].w; }
        }
        acc.x += gw[j] * e.x; acc.y += gw[j] * e.y; acc.z += gw[j] * e.z; acc.w += gw[j] * e.w;
    }
    bf16x4 o;
    o[0] = (bf16)acc.x; o[1] = (bf16)acc.y; o[2] = (bf16)acc.z; o[3] = (bf16)acc.w;
    *reinterpret_cast<bf16x4*>(y + row * d + c) = o;
}

int launch_moe_combine_partials(compact_ctx* ctx, const float* partials, int ks, int64_t total_rows, const float* h,
                                const int32_t* slot_of, const float* sorted_gate, int64_t rows, void* y, hipStream_t s) {
    if (rows == 0) return COMPACT_OK;
    const compact_layer_cfg& c = ctx->cfg;
    dim3 grid((c.d_model / 4 + 255) / 256, (unsigned)rows);
    moe_combine_partials_kernel<<<grid, 256, 0, s>>>(partials, ks, total_rows, h, slot_of, sorted_gate, c.top_k, c.d_model,
                                                     (bf16*)y);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
