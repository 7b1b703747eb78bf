// fp32 GEMM of the fp32 storage mode: C[M,N] = A[M,K] B[N,K]^T (+ R), fp32
// products and sums on the matrix cores (v_mfma_f32_16x16x4_f32).
//
// The mode's layers are small, so what bounds a call is latency: a decode step
// multiplies a handful of rows with a few hundred weight rows.  Hence small
// output tiles (16 x 16, 32 x 32 where those would be thousands, 64 x 64 in large
// calls) whose wavefronts split K: wavefront w takes the 16-wide k-chunks w, w + WAVES, ...,
// loads both operands straight from memory (16 bytes per lane, two to eight
// chunks in flight) and the partial tiles are added in wavefront order through LDS.  The
// split depends on K alone, so a row's bits do not depend on how many rows share
// the call.  Before (64 x 64 tiles, one sequence over K): 4 rows x 256 columns,
// K 1024, 60 us.
#include <type_traits>

#include "vecio.h"

#define F32_CHUNK 16   // k per chunk: one float4 per lane, four MFMAs

struct F32Gemm {
    const float *A, *B, *R;
    float* C;
    int64_t M;
    int N, K;
    int vec;   // rows are 16-byte aligned and K is a multiple of F32_CHUNK
    // front half of an RMSNorm (null norm_g: off): the operand is x * norm_g, the row's result is scaled by 1 / rms(x)
    const float* norm_g;
    float norm_eps;
    GroupedArgs g;
};

// Wavefront w's share of MT x NB output tiles (rows arow[], weight rows brow[] of the lane), and with a norm its share of the
// rows' sums of squares.  UN: chunks in flight, whose loads go out in one batch.
template <int MT, int NB, int WAVES, int UN>
__device__ __forceinline__ void accumulate(const F32Gemm& p, const float* const (&arow)[MT], const float* const (&brow)[NB], int w,
                                           int c, floatx4 (&acc)[MT][NB], float (&ss)[MT]) {
    // lane (r, c) holds k = 16 q + 4 c .. + 3 of row r: MFMA e takes element e of every lane, so a chunk's products are
    // added in the order k = e, 4 + e, 8 + e, 12 + e, the same for both operands
    auto load = [&](const float* row, int q) {
        const int k = q * F32_CHUNK + c * 4;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k + e < p.K) v[e] = row[k + e];
        return v;
    };
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        ss[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int nq = (p.K + F32_CHUNK - 1) / F32_CHUNK;
    auto trip = [&](int q0, auto whole) __attribute__((always_inline)) {   // whole: all of the batch lies inside K
        constexpr bool WHOLE = decltype(whole)::value;
        floatx4 av[UN][MT], bv[UN][NB], gv[UN];
        if (p.vec) {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if (!WHOLE && q0 + u * WAVES >= nq) break;
                const int k = (q0 + u * WAVES) * F32_CHUNK + c * 4;
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[u][j] = *reinterpret_cast<const floatx4*>(brow[j] + k);
                if (p.norm_g) gv[u] = *reinterpret_cast<const floatx4*>(p.norm_g + k);
#pragma unroll
                for (int i = 0; i < MT; ++i) av[u][i] = *reinterpret_cast<const floatx4*>(arow[i] + k);
            }
        } else {
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int q = q0 + u * WAVES;
#pragma unroll
                for (int i = 0; i < MT; ++i) av[u][i] = load(arow[i], q);
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[u][j] = load(brow[j], q);
                if (p.norm_g) gv[u] = load(p.norm_g, q);
            }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            if (!WHOLE && q0 + u * WAVES >= nq) break;
            if (p.norm_g) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        ss[i] = fmaf(av[u][i][e], av[u][i][e], ss[i]);
                        av[u][i][e] *= gv[u][e];
                    }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][i][e], bv[u][j][e], acc[i][j], 0, 0, 0);
        }
    };
    int q0 = w;
    for (; q0 + (UN - 1) * WAVES < nq; q0 += UN * WAVES) trip(q0, std::true_type{});
    if (q0 < nq) trip(q0, std::false_type{});   // (asking for the last chunk again where there is none: K 1152, 512 x 1024 43.5 us)
}

// EPI 0: C = acc (+R).  EPI 1: B is [2N, K] (gate rows then up rows); C = silu(A Bg^T) * (A Bu^T).
// With a GroupedArgs map, row tile blockIdx.y covers rows tile_row0 .. +tile_rows of the expert-sorted order, reads A
// rows through a_gather and uses expert tile_expert's slice of B.
// UN: chunks in flight.  BATCH: their loads in one batch (accumulate()), or each behind a test of its own, with zeros past K.  The
// sums are the same.  launch_f32 says which form is taken where.
template <int EPI, int MT, int NT, int WAVES, int UN, bool BATCH>
__global__ __launch_bounds__(WAVES * 64) void gemm_f32_kernel(const F32Gemm p) {
    constexpr int NB = EPI == 1 ? 2 * NT : NT;   // column tiles of B (SwiGLU: gate tiles, then up tiles)
    constexpr int PT = MT > 2 ? 1 : MT;          // row tiles that are added up at a time
    __shared__ floatx4 part[WAVES][PT * NB][64];
    __shared__ float ssq[WAVES][MT * 16];
    const int lane = threadIdx.x & 63, w = BATCH ? wave_index() : (int)(threadIdx.x >> 6);
    const int r = lane & 15, c = lane >> 4;
    int64_t m0 = (int64_t)blockIdx.y * 16 * MT, m_end = p.M;
    const float* B = p.B;
    if (p.g.tile_expert) {
        const int e = p.g.tile_expert[blockIdx.y];
        if (e < 0) return;
        m0 = p.g.tile_row0[blockIdx.y];
        m_end = m0 + p.g.tile_rows[blockIdx.y];
        B += (int64_t)e * p.g.b_expert_stride;
    }
    const int n0 = blockIdx.x * 16 * NT;
    const float *arow[MT], *brow[NB];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        int64_t m = m0 + i * 16 + r;
        m = m < m_end ? m : m_end - 1;
        arow[i] = p.A + (p.g.a_gather ? (int64_t)p.g.a_gather[m] : m) * p.K;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) brow[j] = B + (int64_t)(min(n0 + (j % NT) * 16 + r, p.N - 1) + (j / NT) * p.N) * p.K;
    floatx4 acc[MT][NB];
    float ss[MT];
    if constexpr (BATCH) {
        accumulate<MT, NB, WAVES, UN>(p, arow, brow, w, c, acc, ss);
    } else {
        // (this loop in a function of its own: other registers, and 20 % of the time of large products more)
        auto load = [&](const float* row, int q) {
            const int k = q * F32_CHUNK + c * 4;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (p.vec) {
                if (k < p.K) v = *reinterpret_cast<const floatx4*>(row + k);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < p.K) v[e] = row[k + e];
            }
            return v;
        };
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            ss[i] = 0.f;
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        const int nq = (p.K + F32_CHUNK - 1) / F32_CHUNK;
        for (int q0 = w; q0 < nq; q0 += UN * WAVES) {
            floatx4 av[UN][MT], bv[UN][NB], gv[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int q = q0 + u * WAVES;
#pragma unroll
                for (int i = 0; i < MT; ++i) av[u][i] = load(arow[i], q);
#pragma unroll
                for (int j = 0; j < NB; ++j) bv[u][j] = load(brow[j], q);
                if (p.norm_g) gv[u] = load(p.norm_g, q);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if (p.norm_g) {
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            ss[i] = fmaf(av[u][i][e], av[u][i][e], ss[i]);
                            av[u][i][e] *= gv[u][e];
                        }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u][i][e], bv[u][j][e], acc[i][j], 0, 0, 0);
            }
        }
    }
    if (p.norm_g) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            ss[i] += __shfl_xor(ss[i], 16, 64);
            ss[i] += __shfl_xor(ss[i], 32, 64);
            if (c == 0) ssq[w][i * 16 + r] = ss[i];
        }
    }
    if constexpr (MT == 1 && NT == 1) {
        // one output per thread: few rows make latency, so the square root, the division and the exponential of an output
        // run beside those of the others
#pragma unroll
        for (int j = 0; j < NB; ++j) part[w][j][lane] = acc[0][j];
        const int row = threadIdx.x >> 4, n = n0 + (threadIdx.x & 15);
        const int64_t m = m0 + row;
        const bool finish = threadIdx.x < 256 && m < m_end && n < p.N;
        float res = 0.f;
        if (EPI == 0 && finish && p.R) res = p.R[m * p.N + n];
        __syncthreads();
        if (!finish) return;
        // output (row, column) is element row % 4 of lane (column, row / 4)
        const int from = (row >> 2) * 16 + (threadIdx.x & 15), e = row & 3;
        float o = part[0][0][from][e], u = part[0][NB - 1][from][e];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) {
            o += part[k][0][from][e];
            u += part[k][NB - 1][from][e];
        }
        if (p.norm_g) {
            float s = ssq[0][row];
#pragma unroll
            for (int k = 1; k < WAVES; ++k) s += ssq[k][row];
            const float rinv = 1.0f / sqrtf(s / (float)p.K + p.norm_eps);
            o *= rinv;
            u *= rinv;
        }
        if (EPI == 1)
            o = o / (1.0f + expf(-o)) * u;
        else if (p.R)
            o += res;
        if (p.g.row_scale) o *= p.g.row_scale[m];
        p.C[m * p.N + n] = o;
        return;
    }
#pragma unroll
    for (int i0 = 0; i0 < MT; i0 += PT) {
        if (i0 > 0) __syncthreads();   // the row tiles before have been read
#pragma unroll
        for (int i = 0; i < PT; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) part[w][i * NB + j][lane] = acc[i0 + i][j];
        __syncthreads();
        // output tile x (row tile x / NT, column tile x % NT) is finished by wavefront x % WAVES; lane (r, c) holds column
        // n0 + 16 j + r of rows m0 + 16 i + 4 c + e
        for (int x = w; x < PT * NT; x += WAVES) {
            const int i = x / NT, j = x % NT;
            auto total = [&](int tile) {
                floatx4 v = part[0][tile][lane];
#pragma unroll
                for (int k = 1; k < WAVES; ++k) {
                    const floatx4 o = part[k][tile][lane];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += o[e];
                }
                return v;
            };
            floatx4 v = total(i * NB + j), u = v;
            if (EPI == 1) u = total(i * NB + NT + j);
            const int n = n0 + j * 16 + r;
            if (n >= p.N) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = (i0 + i) * 16 + 4 * c + e;
                const int64_t m = m0 + row;
                if (m >= m_end) continue;
                float o = v[e];
                if (p.norm_g) {
                    float s = ssq[0][row];
#pragma unroll
                    for (int k = 1; k < WAVES; ++k) s += ssq[k][row];
                    const float rinv = 1.0f / sqrtf(s / (float)p.K + p.norm_eps);
                    o *= rinv;
                    u[e] *= rinv;
                }
                if (EPI == 1)
                    o = o / (1.0f + expf(-o)) * u[e];
                else if (p.R)
                    o += p.R[m * p.N + n];
                if (p.g.row_scale) o *= p.g.row_scale[m];
                p.C[m * p.N + n] = o;
            }
        }
    }
}

// Decode rows: RMSNorm, q/k/v projection, rotation and cache append in one kernel.  A workgroup is two groups of WAVES
// wavefronts: columns i0 .. i0 + 15 of a head and the HD / 2 columns further that they are rotated with.  Sums, factors and
// rotation are those of gemm_f32_kernel and of the decode epilogue (norm_rope.hip), so a row has the same bits either way;
// the angles are formed before the sums.  Bound: latency, the launch that it saves was 2.7 of a step's 28 us (d 256).
struct F32QkvOut {
    const BlockMeta* meta;
    float *q, *k, *v;
    int step, Hq, Hkv, hd;
    double log2_theta;
};
// SINE: wavefronts beside the two groups that form the angles (0: the first of group 0, after their sums).
template <int WAVES, int SINE>
__global__ __launch_bounds__((2 * WAVES + SINE) * 64) void qkv_rope_f32_kernel(const F32Gemm p, const F32QkvOut o) {
    __shared__ floatx4 part[2 * WAVES][64];
    __shared__ float2 angle[256];
    __shared__ float ssq[WAVES][16];
    const int lane = threadIdx.x & 63, w = wave_index();
    const int grp = w / WAVES, wg = w % WAVES;
    const int r = lane & 15, c = lane >> 4;
    const int per_head = o.hd / 32, head = blockIdx.x / per_head, i0 = blockIdx.x % per_head * 16;
    const int m0 = blockIdx.y * 16;
    // thread t < 256 finishes row m0 + t / 16, elements i0 + t % 16 and o.hd / 2 further
    const int row = (threadIdx.x & 255) >> 4, m = min(m0 + row, (int)p.M - 1), col = i0 + (threadIdx.x & 15);
    const bool finish = threadIdx.x < 256 && m0 + row < p.M;
    const BlockMeta bm = o.meta[m];
    auto form_angle = [&]() {
        if (m0 + row >= p.M || head >= o.Hq + o.Hkv) return;
        const double inv_freq = exp2(-2.0 * (double)col / (double)o.hd * o.log2_theta);
        double sn, cn;
        sincos((double)(bm.pos_offset + bm.len + o.step) * inv_freq, &sn, &cn);
        angle[threadIdx.x & 255] = make_float2((float)cn, (float)sn);
    };
    if (w >= 2 * WAVES) {
        form_angle();
    } else {
        const float* arow[1] = {p.A + (int64_t)min(m0 + r, (int)p.M - 1) * p.K};
        const float* brow[1] = {p.B + (int64_t)(head * o.hd + grp * (o.hd / 2) + i0 + r) * p.K};
        floatx4 acc[1][1];
        float ss[1];
        accumulate<1, 1, WAVES, 4>(p, arow, brow, wg, c, acc, ss);
        ss[0] += __shfl_xor(ss[0], 16, 64);
        ss[0] += __shfl_xor(ss[0], 32, 64);
        if (grp == 0 && c == 0) ssq[wg][r] = ss[0];
        part[w][lane] = acc[0][0];
        if (SINE == 0 && threadIdx.x < 256) form_angle();
    }
    __syncthreads();
    if (!finish) return;
    float s = ssq[0][row];
#pragma unroll
    for (int k = 1; k < WAVES; ++k) s += ssq[k][row];
    const float rinv = 1.0f / sqrtf(s / (float)p.K + p.norm_eps);
    // output (row, column) of a tile is element row % 4 of lane (column, row / 4)
    const int from = (row >> 2) * 16 + (threadIdx.x & 15), e = row & 3;
    float lo = part[0][from][e], up = part[WAVES][from][e];
#pragma unroll
    for (int k = 1; k < WAVES; ++k) {
        lo += part[k][from][e];
        up += part[WAVES + k][from][e];
    }
    lo *= rinv;
    up *= rinv;
    const int pos = bm.len + o.step;
    if (head < o.Hq + o.Hkv) {
        float olo, ohi;
        rotate(lo, up, angle[threadIdx.x].x, angle[threadIdx.x].y, olo, ohi);
        float* dst = head < o.Hq ? o.q + ((int64_t)m * o.Hq + head) * o.hd
                                 : o.k + bm.slab + ((int64_t)(head - o.Hq) * bm.capacity + pos) * o.hd;
        dst[col] = olo;
        dst[o.hd / 2 + col] = ohi;
    } else {
        float* vcol = o.v + bm.slab + (int64_t)(head - o.Hq - o.Hkv) * o.hd * bm.capacity + pos;
        vcol[(int64_t)col * bm.capacity] = lo;
        vcol[(int64_t)(o.hd / 2 + col) * bm.capacity] = up;
    }
}

// Covers what the 16 x 16 tiles of launch_f32 cover; beyond that larger tiles and a launch of its own for the rotation.
bool qkv_rope_f32_supported(const compact_layer_cfg& c, int rows) {
    const int64_t cols = (int64_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
    return c.dtype == COMPACT_FP32 && (rows + 15) / 16 * (cols / 16) <= 2048;
}

int launch_qkv_rope_f32(compact_ctx* ctx, const BlockMeta* d_meta, int rows, int step, const float* x, const float* g,
                        const float* w_qkv, float* q, float* d_k, float* d_v, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    if (!qkv_rope_f32_supported(c, rows)) return set_err(ctx, COMPACT_ESHAPE, "fused q/k/v decode kernel does not cover this shape");
    F32Gemm p{};
    p.A = x;
    p.B = w_qkv;
    p.M = rows;
    p.N = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
    p.K = c.d_model;
    p.vec = p.K % F32_CHUNK == 0 && (((uintptr_t)x | (uintptr_t)w_qkv | (uintptr_t)g) & 15) == 0;
    p.norm_g = g;
    p.norm_eps = c.rms_eps;
    const F32QkvOut o{d_meta, q, d_k, d_v, step, c.n_q_heads, c.n_kv_heads, c.head_dim, log2((double)c.rope_theta)};
    const dim3 grid(p.N / 32, (rows + 15) / 16);
    if (p.K >= 1024)
        qkv_rope_f32_kernel<8, 0><<<grid, 1024, 0, s>>>(p, o);
    else
        qkv_rope_f32_kernel<4, 4><<<grid, 768, 0, s>>>(p, o);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

int gemm_f32_mtile() { return 32; }

template <int EPI, int WAVES>
static int launch_f32(compact_ctx* ctx, const F32Gemm& p, bool grouped, hipStream_t s) {
    // 16 x 16 tiles fill the chip with few of them; beyond 2048 (eight per compute unit) 32 x 32 reads half the operands, and
    // from one 64 x 64 tile per compute unit on these read a quarter (160 of them: 28.9 against 30.8 us at N 1024, K 1024;
    // 220: 37.5 against 31.4; 4096 x 4096 x 4096: 2132 -> 1360 us).  SwiGLU holds two operand tiles, so its big tiles are 64 x 32
    // and pay for themselves over a long K only (1024: 106 against 116 us for 880 tiles, 333 against 327 for 2816; 4096^3: 4413
    // -> 2908 us).
    const int64_t small_tiles = (p.M + 15) / 16 * ((p.N + 15) / 16);
    constexpr int BN = EPI == 1 ? 32 : 64;   // columns of a big tile
    const int64_t big_tiles = (p.M + 63) / 64 * ((p.N + BN - 1) / BN);
    const dim3 small((p.N + 15) / 16, (unsigned)((p.M + 15) / 16)), big((p.N + BN - 1) / BN, (unsigned)((p.M + 63) / 64));
    const dim3 middle((p.N + 31) / 32, grouped ? (unsigned)p.g.n_mtiles : (unsigned)((p.M + 31) / 32));
    constexpr int T = WAVES * 64;
    // Loads in one batch (the last one of a wavefront holds what is left) or each behind a test of its own, as measured (us, the
    // form not taken -> the one taken):
    // - 16 x 16 and 32 x 32 tiles: in a batch (512 x 1024, K 320: 13.0 -> 11.1; 600 x 960, K 512: 16.8 -> 14.5; SwiGLU 1024 x
    //   1024, K 512: 39.4 -> 29.2); 16 x 16 over K >= 1024 eight chunks at once while there is one tile per compute unit
    //   (64 x 960, K 1408: 8.2 -> 7.8), four with more;
    // - 64 x 64 tiles: in a batch up to K 2048 (1500 x 1024, K 1152: 64.0 -> 55.7; K 2048 0 .. 7 %), beyond one by one (560 x
    //   1920, K 2880: 133.1 -> 126.6), and so over two chunks in more than one round (1500 x 1024, K 128: 12.0 -> 11.1);
    // - SwiGLU's 64 x 32, which start at K 2048: one by one (560 x 1920, K 2880: 204.6 -> 192.7).
    if (!grouped && small_tiles <= 2048) {
        constexpr int UN = EPI == 0 && WAVES == 8 ? 8 : 4;
        if (UN == 8 && small_tiles <= 256)
            gemm_f32_kernel<EPI, 1, 1, WAVES, UN, true><<<small, T, 0, s>>>(p);
        else
            gemm_f32_kernel<EPI, 1, 1, WAVES, 4, true><<<small, T, 0, s>>>(p);
    } else if (!grouped && big_tiles >= 256 && (EPI == 0 || p.K >= 2048)) {
        const int chunks = p.K / (F32_CHUNK * WAVES);   // of a wavefront, at least
        if (EPI == 0 && p.K <= 2048 && !(WAVES == 4 && chunks == 2 && big_tiles > 256))
            gemm_f32_kernel<EPI, 4, BN / 16, WAVES, 2, EPI == 0><<<big, T, 0, s>>>(p);
        else
            gemm_f32_kernel<EPI, 4, BN / 16, WAVES, 2, false><<<big, T, 0, s>>>(p);
    } else {
        gemm_f32_kernel<EPI, 2, 2, WAVES, EPI == 1 ? 2 : 4, true><<<middle, T, 0, s>>>(p);
    }
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

int launch_gemm_f32(compact_ctx* ctx, const float* A, const float* B, const float* R, float* C, int64_t M, int N,
                    int K, int epilogue, const GroupedArgs* grouped, hipStream_t s, const float* norm_g) {
    if (M == 0) return COMPACT_OK;
    F32Gemm p{};
    p.A = A;
    p.B = B;
    p.R = epilogue == 1 ? nullptr : R;
    p.C = C;
    p.M = M;
    p.N = N;
    p.K = K;
    p.vec = K % F32_CHUNK == 0 && (((uintptr_t)A | (uintptr_t)B | (uintptr_t)norm_g) & 15) == 0;
    p.norm_g = norm_g;
    p.norm_eps = ctx->cfg.rms_eps;
    if (grouped) p.g = *grouped;
    // wavefronts per tile by K alone: at least eight k-chunks each
    if (epilogue == 1) return K >= 1024 ? launch_f32<1, 8>(ctx, p, grouped != nullptr, s) : launch_f32<1, 4>(ctx, p, grouped != nullptr, s);
    return K >= 1024 ? launch_f32<0, 8>(ctx, p, grouped != nullptr, s) : launch_f32<0, 4>(ctx, p, grouped != nullptr, s);
}
