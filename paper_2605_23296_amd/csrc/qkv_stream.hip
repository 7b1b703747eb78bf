// q/k/v projection of a decode step (bf16 storage, at most 64 rows) with the RMSNorm before it and the rotary embedding
// and the cache append behind it: one launch, nothing written but the rotated query rows, the K rows and the V columns.
//
//  * a workgroup owns P groups of 8 weight rows and all of K; wavefront w streams the w-th slice of 512 k through a
//    ring of its own in LDS, pieces of 8 rows x 128 bytes (see gemv_stream.hip: whole lines, landing in LDS directly,
//    no barrier before the sums);
//  * a group is 4 rows of a head's lower half and the 4 rows that rotate with them, so both elements of a pair end up
//    in one wavefront, 16 lanes apart; two groups are an MFMA tile;
//  * x arrives as it is: bf16(x g) is formed on the operand fragment, the sum of x^2 of a row from the same registers;
//  * the angles (64 bits) are formed by two wavefronts of their own beside the stream (by all, behind it, where 16 stream);
//  * slices, the order of the MFMA steps inside one, the order in which slices are added and the tree of a row's
//    sum of squares are those of gemm_skinny_kernel and decode_qkv_epilogue_kernel, which serve the steps that
//    qkv_stream_supported() leaves out: a row has the same bits there.
// 6144 x 4096 at 8 / 24 / 64 rows: 12.0 + 4.5 / 15.7 + 5.1 / 21.5 + 7.2 us (split-K projection and epilogue) -> 12.3 / 15.0 / 19.3;
// 5120 x 2880 at 16 rows 10.1 us.  50 MB at 6.1 TB/s, what a long stream of such loads reaches, would be 8.2 us; the rest is the
// first loads' way, the sums and the activation rows, which every workgroup reads (64 rows,
// three groups per workgroup instead of six: 24.6 us).  At 8 rows two tiles of 16 weight rows per workgroup (192
// workgroups) and the angles in the streaming wavefronts: 15.0 us.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "stream_lds.h"
#include "vecio.h"

#define QS_SLICE 512
#define QS_UNITS (QS_SLICE / 64)
#define QS_MAX_WAVES 16
#define QS_ANGLE_WAVES 2

struct QkvStreamArgs {
    const bf16 *X, *W, *g;
    int M, K, n_groups;
    int Hq, Hkv, hd, step;
    const BlockMeta* meta;
    bf16 *q, *k, *v;
    double log2_theta;
    float inv_d, eps;
};

// Waits for all but the loads of the n <= N youngest units.
template <int NL, int N>
__device__ __forceinline__ void wait_behind(int n) {
    if constexpr (N == 0)
        gs_wait<0>();
    else if (n >= N)
        gs_wait<N * NL>();
    else
        wait_behind<NL, N - 1>(n);
}

// P: groups per workgroup.  XI: 8-row pieces of activations (rows / 8).  D: units (64 k of the groups and of the rows) in a
// wavefront's ring.
template <int P, int XI, int D>
struct QkvStreamShape {
    static constexpr int LOADS = P + XI;   // per unit, 1 KB each
    static constexpr int T = (P + 1) / 2, MT = (XI + 1) / 2;
    static constexpr int RING = (D * LOADS + 1) * 1024, RED = T * MT * 1024;
    static constexpr int AREA = RING > RED ? RING : RED;        // of a wavefront: ring and its slice of g, later partial tiles
    static constexpr int ANGLES = P * XI * 8 * 4;
    static int smem(int slices) { return slices * (AREA + XI * 8 * 4) + ANGLES * 8; }
};

template <int P, int XI, int D>
__global__ __launch_bounds__(QS_MAX_WAVES * 64) void qkv_stream_kernel(QkvStreamArgs p, const int slices) {
    typedef QkvStreamShape<P, XI, D> Shape;
    constexpr int T = Shape::T, MT = Shape::MT, NL = Shape::LOADS, R = XI * 8;
    {   // rows of this workgroup
        const int m0 = blockIdx.y * R;
        p.M = min(p.M - m0, R);
        p.X += (size_t)m0 * p.K;
        p.meta += m0;
        p.q += (size_t)m0 * p.Hq * p.hd;
    }
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, w = wave_index(), waves = blockDim.x >> 6;
    const int r = lane & 15, c = lane >> 4, lrow = lane >> 3;
    float2* const angle = reinterpret_cast<float2*>(smem + slices * Shape::AREA);                   // [P][R][4]
    float* const ssq = reinterpret_cast<float*>(smem + slices * Shape::AREA + Shape::ANGLES * 8);   // [slices][R]
    const int group0 = blockIdx.x * P, per_head = p.hd / 8, half = p.hd / 2;

    // angles of thread t0 of nt
    auto form_angles = [&](int t0, int nt) {
        for (int a = t0; a < Shape::ANGLES; a += nt) {
            const int row = (a >> 2) % R, group = group0 + (a >> 2) / R;
            if (row >= p.M || group >= p.n_groups || group / per_head >= p.Hq + p.Hkv) continue;
            const double inv_freq = exp2(-2.0 * (double)(group % per_head * 4 + (a & 3)) / (double)p.hd * p.log2_theta);
            double sn, cn;
            sincos((double)(p.meta[row].pos_offset + p.meta[row].len + p.step) * inv_freq, &sn, &cn);
            angle[a] = make_float2((float)cn, (float)sn);
        }
    };

    floatx4 acc[T][MT];
    if (w >= slices) {
        form_angles(threadIdx.x - slices * 64, (waves - slices) * 64);
    } else {
        char* const ring = smem + w * Shape::AREA;
        char* const gs = ring + D * NL * 1024;
        const int k0 = w * QS_SLICE, klen = min(QS_SLICE, p.K - k0), units = klen / 64;
        // lane l of a load: row l / 8 of 8, LDS position l % 8; piece i is row i * 8 + l / 8 of its tile, group q the half q % 2
        const bf16* wsrc[P];
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const int group = min(group0 + q, p.n_groups - 1);
            const int n = group / per_head * p.hd + group % per_head * 4 + (lrow & 3) + (lrow >> 2) * half;
            wsrc[q] = p.W + (size_t)n * p.K + k0 + ((lane & 7) ^ ((((q & 1) * 8 + lrow) >> 1) & 7)) * 8;
        }
        const bf16* xsrc[XI];
#pragma unroll
        for (int i = 0; i < XI; ++i)
            xsrc[i] = p.X + (size_t)min(i * 8 + lrow, p.M - 1) * p.K + k0 + ((lane & 7) ^ (((i * 8 + lrow) >> 1) & 7)) * 8;
        auto issue = [&](int u, int slot) {
            char* const dst = ring + slot * NL * 1024;
#pragma unroll
            for (int i = 0; i < XI; ++i) load16_to_lds(xsrc[i] + u * 64, dst + i * 1024);
#pragma unroll
            for (int q = 0; q < P; ++q) load16_to_lds(wsrc[q] + u * 64, dst + (XI + q) * 1024);
        };
        load16_to_lds(p.g + k0 + min(lane, klen / 8 - 1) * 8, gs);
#pragma unroll
        for (int u = 0; u < D; ++u)
            if (u < units) issue(u, u);

        // LDS offsets of the operand fragments of k-step h: row r, chunk 4 h + c
        int foff[2], fodd[2], xoff[MT][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            foff[h] = r * 128 + (((4 * h + c) ^ ((r >> 1) & 7)) << 4);
            fodd[h] = (r & 7) * 128 + (((4 * h + c) ^ ((r & 7) >> 1)) << 4);   // (a tile of one group: its rows twice)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int xr = min(mt * 16 + r, R - 1);   // (columns beyond the rows are not read by anybody)
                xoff[mt][h] = xr * 128 + (((4 * h + c) ^ ((xr >> 1) & 7)) << 4);
            }
        }
        float sq[MT][QS_UNITS][2];   // sums of x^2 over 8 elements
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < QS_UNITS; ++u) sq[mt][u][0] = sq[mt][u][1] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < QS_UNITS; ++u)
            if (u < units) {
                wait_behind<NL, D - 1>(min(u + D, units) - u - 1);   // the units behind this one may still fly
                const char* const src = ring + (u % D) * NL * 1024;
                bf16x8 xf[MT][2], wf[T][2], gf[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    gf[h] = *reinterpret_cast<const bf16x8*>(gs + ((u * 8 + 4 * h + c) << 4));
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) xf[mt][h] = *reinterpret_cast<const bf16x8*>(src + xoff[mt][h]);
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        wf[t][h] = *reinterpret_cast<const bf16x8*>(src + (XI + 2 * t) * 1024 + (2 * t + 1 < P ? foff[h] : fodd[h]));
                }
                gs_lds_done();   // the slot may be filled again
                if (u + D < QS_UNITS && u + D < units) issue(u + D, u % D);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        float ss = 0.f;
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const float f = (float)xf[mt][h][j];
                            ss += f * f;
                            xf[mt][h][j] = (bf16)(f * (float)gf[h][j]);
                        }
                        sq[mt][u][h] = ss;
#pragma unroll
                        for (int t = 0; t < T; ++t)
                            acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t][h], xf[mt][h], acc[t][mt], 0, 0, 0);
                    }
            }
        // the butterfly over the 64 pieces of a row's slice: piece 8 u + 4 h + c
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int o = QS_UNITS / 2; o > 0; o >>= 1)
#pragma unroll
                for (int u = 0; u < o; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) sq[mt][u][h] += sq[mt][u + o][h];
            float ss = sq[mt][0][0] + sq[mt][0][1];
            ss += __shfl_xor(ss, 32, 64);
            ss += __shfl_xor(ss, 16, 64);
            if (c == 0 && mt * 16 + r < R) ssq[w * R + mt * 16 + r] = ss;
        }
        // the wavefront's own ring is dead: its partial tiles take its place
        floatx4* const red = reinterpret_cast<floatx4*>(ring);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) red[(t * MT + mt) * 64 + lane] = acc[t][mt];
        if (waves == slices) form_angles(threadIdx.x, blockDim.x);
    }
    __syncthreads();
    for (int f = w; f < T * MT; f += waves) {
        const int t = f / MT, row = f % MT * 16 + r, q = 2 * t + (c >> 1), group = group0 + q;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        float ss = 0.f;
        for (int s = 0; s < slices; ++s) {
            const floatx4 o = reinterpret_cast<const floatx4*>(smem + s * Shape::AREA)[f * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += o[e];
            ss += ssq[s * R + min(row, R - 1)];
        }
        const float rinv = 1.0f / sqrtf(ss * p.inv_d + p.eps);
        // lanes with even c: elements i .. i + 3 of the lower half, odd: their partners
        float other[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] *= rinv;
            other[e] = __shfl_xor(v[e], 16, 64);
        }
        if (row >= p.M || q >= P || group >= p.n_groups) continue;
        const bool upper = c & 1;
        const int head = group / per_head, n = group % per_head * 4 + (upper ? half : 0);
        const BlockMeta bm = p.meta[row];
        const int at = bm.len + p.step;
        if (head < p.Hq + p.Hkv) {
            bf16x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 cs = angle[(q * R + row) * 4 + e];
                float lo, hi;
                rotate(upper ? other[e] : v[e], upper ? v[e] : other[e], cs.x, cs.y, lo, hi);
                out[e] = (bf16)(upper ? hi : lo);
            }
            bf16* const dst = head < p.Hq ? p.q + ((size_t)row * p.Hq + head) * p.hd
                                          : p.k + bm.slab + ((size_t)(head - p.Hq) * bm.capacity + at) * p.hd;
            *reinterpret_cast<bf16x4*>(dst + n) = out;
        } else {
            bf16* const vcol = p.v + bm.slab + (size_t)(head - p.Hq - p.Hkv) * p.hd * bm.capacity + at;
#pragma unroll
            for (int e = 0; e < 4; ++e) vcol[(size_t)(n + e) * bm.capacity] = (bf16)v[e];
        }
    }
}

#define QS_LDS (160 * 1024)
template <int P, int XI, int D>
static int launch_qs_cfg(compact_ctx* ctx, const QkvStreamArgs& p, int slices, hipStream_t s) {
    auto kern = qkv_stream_kernel<P, XI, D>;
    static bool attr = false;
    if (!attr) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, QS_LDS));
        attr = true;
    }
    const int waves = std::min(slices + QS_ANGLE_WAVES, QS_MAX_WAVES);
    kern<<<dim3((p.n_groups + P - 1) / P, (p.M + XI * 8 - 1) / (XI * 8)), waves * 64, QkvStreamShape<P, XI, D>::smem(slices), s>>>(p, slices);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
// the deepest ring that fits
template <int P, int XI>
static int launch_qs_depth(compact_ctx* ctx, const QkvStreamArgs& p, int slices, hipStream_t s) {
    if constexpr (P == 1 && XI <= 2)
        if (QkvStreamShape<P, XI, 8>::smem(slices) <= QS_LDS) return launch_qs_cfg<P, XI, 8>(ctx, p, slices, s);
    if (QkvStreamShape<P, XI, 3>::smem(slices) <= QS_LDS) return launch_qs_cfg<P, XI, 3>(ctx, p, slices, s);
    if (QkvStreamShape<P, XI, 2>::smem(slices) <= QS_LDS) return launch_qs_cfg<P, XI, 2>(ctx, p, slices, s);
    if (QkvStreamShape<P, XI, 1>::smem(slices) <= QS_LDS) return launch_qs_cfg<P, XI, 1>(ctx, p, slices, s);
    return set_err(ctx, COMPACT_ESHAPE, "fused q/k/v projection: no ring fits");
}

// 17 .. 64 rows: up to eight slices (the ring of one unit fits for every number of groups).  33 .. 40 rows take two workgroups with
// room for 48; where these need a second round the split-K kernel and its epilogue are faster (whole steps of 33 rows, little beside
// the projection: d 4096, 1024 groups 70.2 us against 72.3, 1792 groups 93.1 against 96.5; d 2880, 1280 groups 65.8 against 69.1;
// at 48 rows both alike), but for short contractions, where launches count (d 1024, 1792 groups: 50.0 against 49.9).
bool qkv_stream_supported(const compact_layer_cfg& c, int rows) {
    const bool one_round = (c.n_q_heads + 2 * c.n_kv_heads) * (c.head_dim / 8) <= 128 * 6;   // two halves, six groups each
    if (rows > 32 && rows <= 40 && !one_round && c.d_model > 1024) return false;
    return c.dtype == COMPACT_BF16 && c.d_model % 64 == 0 && rows >= 1 &&
           (rows <= 16 ? c.d_model <= QS_MAX_WAVES * QS_SLICE : rows <= 64 && c.d_model <= 8 * QS_SLICE);
}

int launch_qkv_stream(compact_ctx* ctx, const BlockMeta* d_meta, int rows, int step, const bf16* x, const bf16* g, const bf16* W,
                      bf16* q, bf16* k, bf16* v, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    if (!qkv_stream_supported(c, rows)) return set_err(ctx, COMPACT_ESHAPE, "fused q/k/v projection does not cover this shape");
    QkvStreamArgs p{};
    p.X = x;
    p.W = W;
    p.g = g;
    p.M = rows;
    p.K = c.d_model;
    p.n_groups = (c.n_q_heads + 2 * c.n_kv_heads) * (c.head_dim / 8);
    p.Hq = c.n_q_heads;
    p.Hkv = c.n_kv_heads;
    p.hd = c.head_dim;
    p.step = step;
    p.meta = d_meta;
    p.q = q;
    p.k = k;
    p.v = v;
    p.log2_theta = log2((double)c.rope_theta);
    p.inv_d = 1.0f / (float)c.d_model;
    p.eps = c.rms_eps;
    const int slices = (c.d_model + QS_SLICE - 1) / QS_SLICE;
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    // More than 32 rows: two workgroups with half of them each read the same weights, one grid row apart.  Workgroups go round the
    // eight XCDs, so the second reading finds them in its XCD's L2 where a grid row is a multiple of 8 workgroups (768 groups: 128
    // of 6 each) and in the cache behind the L2s elsewhere.
    const int halves = rows > 32 ? 2 : 1;
    const int each = (rows + halves - 1) / halves;
    // Groups per workgroup: the rounds of one workgroup per compute unit that cost the fewest loads per unit, of the groups and of
    // the activation rows, more groups where equal.  By the groups alone, 896 of them were one per workgroup beyond 32 rows, seven
    // rounds that asked for four pieces of rows beside each of weights (d 4096, 64 rows: a step 104.9 us, now 74.7), 1792
    // likewise (64 rows 127.7 -> 103.7, 16 rows 79.2 -> 65.3).
    int best = 1;
    int64_t best_cost = 0;
    for (int n : {1, 2, 3, 5, 6}) {
        const int64_t wgs = (int64_t)halves * ((p.n_groups + n - 1) / n), cost = (wgs + n_cus - 1) / n_cus * (n + (each + 7) / 8);
        if (n == 1 || (cost <= best_cost && halves * p.n_groups > n_cus)) {
            best = n;
            best_cost = cost;
        }
    }
    auto go = [&](auto tag) {
        constexpr int P = decltype(tag)::value;
        return each <= 8    ? launch_qs_depth<P, 1>(ctx, p, slices, s)
               : each <= 16 ? launch_qs_depth<P, 2>(ctx, p, slices, s)
               : each <= 24 ? launch_qs_depth<P, 3>(ctx, p, slices, s)
                            : launch_qs_depth<P, 4>(ctx, p, slices, s);
    };
    switch (best) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        case 5: return go(std::integral_constant<int, 5>{});
        default: return go(std::integral_constant<int, 6>{});
    }
}
