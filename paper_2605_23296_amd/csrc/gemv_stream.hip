// Whole-K weight-streaming projections of the decode step (bf16 storage, at most
// 16 activation rows): a workgroup of 16 wavefronts owns T tiles of 16 weight rows,
// so the sum over K is finished inside the kernel and the step that follows the
// projection (residual add + the pieces of the next RMSNorm, SwiGLU, closing
// residual add) is applied before anything is written.  No split-K partials, no
// second launch.
//
//  * what bounds them is the path from memory into the compute unit: it holds about
//    32 KB of requests, and takes as many clocks for a load as there are groups of
//    four lanes that are not one contiguous run.  So every load is 8 rows x 128 bytes
//    (whole lines, 8 lanes to a line) and lands in LDS directly; loads in the order
//    of the MFMA operand (a lane per row, 64-byte pieces) stream 235 MB at 4.2 TB/s,
//    these at 6.1;
//  * wavefront kw takes the 64-wide pieces ("units") kw, kw + 16, ... of K for all T
//    tiles and keeps a ring of its own of D tile pieces (2 KB each) and the
//    activation rows of as many units: no barrier, no wait but its own, so nothing
//    runs in lockstep and the stream does not pause at a stage;
//  * one 128-byte row of activations serves T tiles (the chip-wide grid picks T so
//    that one workgroup per compute unit covers the matrix);
//  * chunks of 16 bytes sit at chunk ^ ((row / 2) % 8) of their row: 16 lanes that
//    read one chunk of 16 rows touch 16 different bank groups, and a lane's global
//    address stays inside the line;
//  * the 16 partial tiles are added in wavefront order through LDS, so the result does
//    not depend on timing or on the batch a row is decoded in.
// 8B-shaped layer at 1 / 8 / 16 rows: gate/up 50.5 / 49.5 / 57.1 -> 45.6 / 45.6 / 47.1 us, output and down projection
// together 32.4 / 37.7 / 44.3 -> 30.2 / 30.8 / 34.9 us (kernels with loads in operand order, activations in LDS for gate/up and
// from L2 for the others); d 1024, FFN 2816, one row: a step 37.5 -> 26.6 us (three launches less).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "stream_lds.h"
#include "vecio.h"

#define GS_WAVES 16
#define GS_MAX_TILES 8

enum StreamStep {
    STREAM_RESID_NORM,   // h = resid + X W^T (fp32), hg = bf16(h * g), ssq_parts[tile][m] = sum over the tile's columns of h^2
    STREAM_RESID_OUT,    // y = bf16(resid_f32 + X W^T)
    STREAM_SWIGLU        // act = silu(r X Wg^T) * (r X Wu^T): a tile is 8 gate rows and the 8 up rows of the same columns
};
struct StreamArgs {
    const bf16 *X, *W;
    int M, N, K, n_tiles;   // N: output columns (SwiGLU: F, W has 2 F rows)
    const bf16 *resid, *g;  // RESID_NORM
    float* h;               // RESID_NORM: out; RESID_OUT: in
    bf16* out;              // hg, y, act
    float* ssq_parts;       // RESID_NORM
    RowNorm norm;           // SWIGLU
};

// XI: 8-row pieces of activations per unit (1: at most 8 rows, 2: at most 16).  D: tile pieces in a wavefront's ring.
template <int T, int XI>
struct StreamShape {
    static constexpr int D = T <= 2 && XI == 2 ? 2 : 3;
    static constexpr int XD = (T - 1 + D) / T;               // units whose activations are in the ring
    static constexpr int XSLOT = XI * 1024, WSLOT = 2048;    // bytes
    static constexpr int WAVE_BYTES = D * WSLOT + XD * XSLOT;
    static constexpr int RED_BYTES = GS_WAVES * T * 64 * 16;
    static constexpr int SMEM = GS_WAVES * WAVE_BYTES > RED_BYTES ? GS_WAVES * WAVE_BYTES : RED_BYTES;
    static_assert(SMEM <= 159 * 1024, "one workgroup per compute unit");
};

template <int T, int XI, StreamStep STEP>
__global__ __launch_bounds__(GS_WAVES * 64) void row_stream_kernel(const StreamArgs p) {
    typedef StreamShape<T, XI> Shape;
    constexpr int D = Shape::D, XD = Shape::XD;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ float rinv[16];
    const int lane = threadIdx.x & 63;
    const int kw = wave_index();
    const int r = lane & 15, c = lane >> 4;
    const int tile0 = blockIdx.x * T;

    // column-group sums of squares of row kw: requested first (the loads land in order), added up behind the stream
    constexpr int PMAX = 8;   // parts per lane (nparts <= 512)
    float pv[PMAX];
    if (STEP == STREAM_SWIGLU) {
#pragma unroll
        for (int u = 0; u < PMAX; ++u) {
            const int pidx = lane + 64 * u;
            pv[u] = kw < p.M && pidx < p.norm.nparts ? p.norm.ssq_parts[(size_t)pidx * p.M + kw] : 0.f;
        }
    }

    // lane l of a load: row l / 8 of 8, LDS position l % 8, hence chunk (l % 8) ^ ((row / 2) % 8) of the row's 128 bytes
    const int lrow = lane >> 3;
    const bf16* wsrc[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = i * 8 + lrow, tile = min(tile0 + t, p.n_tiles - 1);
            int n;   // weight row of tile row `row`
            if (STEP == STREAM_SWIGLU)
                n = i * p.N + min(tile * 8 + lrow, p.N - 1);
            else
                n = min(tile * 16 + row, p.N - 1);
            wsrc[t][i] = p.W + (size_t)n * p.K + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
        }
    const bf16* xsrc[XI];
#pragma unroll
    for (int i = 0; i < XI; ++i) xsrc[i] = p.X + (size_t)min(i * 8 + lrow, p.M - 1) * p.K + ((lane & 7) ^ (((i * 8 + lrow) >> 1) & 7)) * 8;
    char* const wring = smem + kw * Shape::WAVE_BYTES;
    char* const xring = wring + D * Shape::WSLOT;
    const int n_units = p.K / 64;
    const int units = (n_units - kw + GS_WAVES - 1) / GS_WAVES;   // of this wavefront (may be 0)

    auto issue_x = [&](int u, int slot) {
        const int k = (u * GS_WAVES + kw) * 64;
#pragma unroll
        for (int i = 0; i < XI; ++i)
            if (i * 8 + lrow < p.M) load16_to_lds(xsrc[i] + k, xring + slot * Shape::XSLOT + i * 1024);
    };
    auto issue_w = [&](const bf16* const (&src)[2], int u, int slot) {
        const int k = (u * GS_WAVES + kw) * 64;
        load16_to_lds(src[0] + k, wring + slot * Shape::WSLOT);
        load16_to_lds(src[1] + k, wring + slot * Shape::WSLOT + 1024);
    };
    floatx4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    // prologue: tile pieces 0 .. D - 1 (piece q: tile q % T of unit q / T) and the activations of their units
#pragma unroll
    for (int q = 0; q < D; ++q)
        if (q / T < units) {
            if (q % T == 0) issue_x(q / T, q / T);
            issue_w(wsrc[q % T], q / T, q);
        }
    // LDS offsets of the operand fragments of k-step h: row r, chunk 4 h + c
    int foff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) foff[h] = r * 128 + (((4 * h + c) ^ ((r >> 1) & 7)) << 4);
    const int xr = min(r, XI * 8 - 1);   // (columns beyond the rows staged are not read by anybody)
    int xoff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) xoff[h] = xr * 128 + (((4 * h + c) ^ ((xr >> 1) & 7)) << 4);

    int wslot = 0, xslot = 0;   // of the piece and of the unit that come next
    for (int u = 0; u < units; ++u) {
        bf16x8 xf[2];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            // at most the D - 1 younger pieces may still fly (near the end fewer are: wait for all)
            if ((units - u) * T - t >= D)
                gs_wait<2 * (D - 1)>();
            else
                gs_wait<0>();
            if (t == 0) {
#pragma unroll
                for (int h = 0; h < 2; ++h) xf[h] = *reinterpret_cast<const bf16x8*>(xring + xslot * Shape::XSLOT + xoff[h]);
                xslot = xslot + 1 == XD ? 0 : xslot + 1;
            }
            bf16x8 wf[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) wf[h] = *reinterpret_cast<const bf16x8*>(wring + wslot * Shape::WSLOT + foff[h]);
            gs_lds_done();   // the slots may be filled again
            const int nu = u + (t + D) / T;
            if (nu < units) {
                if ((t + D) % T == 0) {
                    // slot of unit nu: XD units after the one whose slot was read last
                    int xs = xslot + ((t + D) / T - 1) % XD;
                    issue_x(nu, xs >= XD ? xs - XD : xs);
                }
                issue_w(wsrc[(t + D) % T], nu, wslot);
            }
            wslot = wslot + 1 == D ? 0 : wslot + 1;
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h], xf[h], acc[t], 0, 0, 0);
        }
    }
    gs_wait<0>();
    if (STEP == STREAM_SWIGLU) {
        float ss = 0.f;   // a fixed summation order: per lane, then a butterfly
#pragma unroll
        for (int u = 0; u < PMAX; ++u) ss += pv[u];
        ss = wave_sum(ss);
        if (lane == 0) rinv[kw] = 1.0f / sqrtf(ss * p.norm.inv_d + p.norm.eps);
    }
    __syncthreads();   // the rings are dead: the partial tiles take their place
    floatx4* red = reinterpret_cast<floatx4*>(smem);   // [GS_WAVES][T][64]
#pragma unroll
    for (int t = 0; t < T; ++t) red[(kw * T + t) * 64 + lane] = acc[t];
    __syncthreads();
    const int tile = tile0 + kw;   // wavefront kw finishes tile kw
    if (kw >= T || tile >= p.n_tiles) return;
    floatx4 v = red[kw * 64 + lane];
#pragma unroll
    for (int w = 1; w < GS_WAVES; ++w) {
        const floatx4 o = red[(w * T + kw) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += o[e];
    }
    // v[e]: activation row r, tile row 4 c + e
    if (STEP == STREAM_SWIGLU) {
        // c < 2: gate of column 4 c + e, c >= 2: up of column 4 (c - 2) + e
        const float rs = rinv[r];
        bf16x4 out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float up = __shfl_xor(v[e], 32, 64) * rs;
            const float g = v[e] * rs;
            out[e] = (bf16)(g / (1.0f + expf(-g)) * up);   // (__expf: off by up to 3.4e-6 of the value at g = -80)
        }
        if (c < 2 && r < p.M) *reinterpret_cast<bf16x4*>(p.out + (size_t)r * p.N + tile * 8 + 4 * c) = out;
    } else if (STEP == STREAM_RESID_OUT) {
        if (r < p.M) {
            const size_t o = (size_t)r * p.N + tile * 16 + 4 * c;
            const floatx4 h = *reinterpret_cast<const floatx4*>(p.h + o);
            bf16x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (bf16)(h[e] + v[e]);
            *reinterpret_cast<bf16x4*>(p.out + o) = out;
        }
    } else {
        float ss = 0.f;
        if (r < p.M) {
            const size_t o = (size_t)r * p.N + tile * 16 + 4 * c;
            const bf16x4 rv = *reinterpret_cast<const bf16x4*>(p.resid + o);
            const bf16x4 gv = *reinterpret_cast<const bf16x4*>(p.g + tile * 16 + 4 * c);
            bf16x4 hg;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] += (float)rv[e];
                hg[e] = (bf16)(v[e] * (float)gv[e]);
                ss += v[e] * v[e];
            }
            *reinterpret_cast<floatx4*>(p.h + o) = v;
            *reinterpret_cast<bf16x4*>(p.out + o) = hg;
        }
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (c == 0 && r < p.M) p.ssq_parts[(size_t)tile * p.M + r] = ss;
    }
}

template <int T, int XI, StreamStep STEP>
static int launch_stream_cfg(compact_ctx* ctx, const StreamArgs& p, hipStream_t s) {
    constexpr int smem = StreamShape<T, XI>::SMEM;
    auto kern = row_stream_kernel<T, XI, STEP>;
    static bool attr = false;
    if (!attr) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        attr = true;
    }
    kern<<<(p.n_tiles + T - 1) / T, GS_WAVES * 64, smem, s>>>(p);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// Tiles per workgroup: the rounds of one workgroup per compute unit that cost the fewest loads, of the tiles and of the
// activation rows (at most GS_MAX_TILES); one per workgroup while that is one round.  The sums of a row do not depend on it.
// By the tiles alone, an FFN of 20544 took one tile per workgroup in eleven rounds, each asking for the rows again (d 5120, 16
// rows: a step 194 us; six tiles, two rounds: 149); one of 25600 and d 5120 likewise (235 -> 176 us).
template <StreamStep STEP>
static int launch_stream(compact_ctx* ctx, const StreamArgs& p, hipStream_t s) {
    if (p.M < 1 || p.M > 16 || p.K % 64 != 0 || p.K < 64 || p.N < 16 || p.N % 16 != 0)
        return set_err(ctx, COMPACT_ESHAPE, "whole-K streaming kernel takes 1..16 rows, N % 16 == 0 and K % 64 == 0");
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    int best = 1;
    int64_t best_cost = 0;
    for (int t = 1; t <= GS_MAX_TILES; ++t) {
        const int64_t wgs = (p.n_tiles + t - 1) / t, cost = (wgs + n_cus - 1) / n_cus * (2 * t + (p.M + 7) / 8);
        if (t == 1 || cost < best_cost) {
            best = t;
            best_cost = cost;
        }
    }
    if (p.n_tiles <= n_cus) best = 1;
    auto go = [&](auto tag) {
        constexpr int T = decltype(tag)::value;
        return p.M <= 8 ? launch_stream_cfg<T, 1, STEP>(ctx, p, s) : launch_stream_cfg<T, 2, STEP>(ctx, p, s);
    };
    switch (best) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        case 4: return go(std::integral_constant<int, 4>{});
        case 5: return go(std::integral_constant<int, 5>{});
        case 6: return go(std::integral_constant<int, 6>{});
        case 7: return go(std::integral_constant<int, 7>{});
        default: return go(std::integral_constant<int, 8>{});
    }
}

int launch_resid_norm_stream(compact_ctx* ctx, const bf16* X, const bf16* W, const bf16* resid, const bf16* g, float* h_out,
                             bf16* hg_out, float* ssq_parts, int M, int N, int K, hipStream_t s) {
    StreamArgs p{};
    p.X = X;
    p.W = W;
    p.M = M;
    p.N = N;
    p.K = K;
    p.n_tiles = N / 16;
    p.resid = resid;
    p.g = g;
    p.h = h_out;
    p.out = hg_out;
    p.ssq_parts = ssq_parts;
    return launch_stream<STREAM_RESID_NORM>(ctx, p, s);
}

int launch_resid_out_stream(compact_ctx* ctx, const bf16* X, const bf16* W, const float* resid, bf16* y, int M, int N, int K,
                            hipStream_t s) {
    StreamArgs p{};
    p.X = X;
    p.W = W;
    p.M = M;
    p.N = N;
    p.K = K;
    p.n_tiles = N / 16;
    p.h = const_cast<float*>(resid);
    p.out = y;
    return launch_stream<STREAM_RESID_OUT>(ctx, p, s);
}

int launch_swiglu_stream(compact_ctx* ctx, const bf16* X, const bf16* W, bf16* act, int M, int F, int K, const RowNorm& norm,
                         hipStream_t s) {
    if (norm.nparts > 512) return set_err(ctx, COMPACT_ESHAPE, "fused gate/up decode kernel takes 512 column groups at most");
    StreamArgs p{};
    p.X = X;
    p.W = W;
    p.M = M;
    p.N = F;
    p.K = K;
    p.n_tiles = F / 8;
    p.out = act;
    p.norm = norm;
    return launch_stream<STREAM_SWIGLU>(ctx, p, s);
}

// m[r][c] = bf16(hg[r][c] / rms_r), 1 / rms from the column sums of squares
__global__ __launch_bounds__(256) void rownorm_apply_kernel(const bf16* __restrict__ hg, const RowNorm norm, bf16* __restrict__ m,
                                                            int rows, int d) {
    __shared__ float s_rinv;
    const int row = blockIdx.x;
    if (threadIdx.x < 64) {
        float ss = 0.f;
        for (int p = threadIdx.x; p < norm.nparts; p += 64) ss += norm.ssq_parts[(size_t)p * rows + row];
        ss = wave_sum(ss);
        if (threadIdx.x == 0) s_rinv = 1.0f / sqrtf(ss * norm.inv_d + norm.eps);
    }
    __syncthreads();
    const float rs = s_rinv;
    for (int c0 = threadIdx.x * 8; c0 < d; c0 += 256 * 8) {
        const bf16x8 v = *reinterpret_cast<const bf16x8*>(hg + (size_t)row * d + c0);
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (bf16)((float)v[j] * rs);
        *reinterpret_cast<bf16x8*>(m + (size_t)row * d + c0) = o;
    }
}

int launch_rownorm_apply(compact_ctx* ctx, const bf16* hg, const RowNorm& norm, bf16* m, int rows, int d, hipStream_t s) {
    rownorm_apply_kernel<<<rows, 256, 0, s>>>(hg, norm, m, rows, d);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
