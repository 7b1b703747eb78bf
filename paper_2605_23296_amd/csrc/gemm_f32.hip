// fp32 GEMM of the fp32 storage mode: C[M,N] = A[M,K] B[N,K]^T (+ R), fp32
// products and sums on the matrix cores (v_mfma_f32_16x16x4_f32).
//
// The mode's layers are small, so what bounds a call is latency: a decode step
// multiplies a handful of rows with a few hundred weight rows.  Hence small
// output tiles (16 x 16, 32 x 32 where those would be thousands, 64 x 64 in large
// calls) whose wavefronts split K: wavefront w takes the 16-wide k-chunks w, w + WAVES, ...,
// loads both operands straight from memory (16 bytes per lane, four chunks in
// flight) and the partial tiles are added in wavefront order through LDS.  The
// split depends on K alone, so a row's bits do not depend on how many rows share
// the call.  Before (64 x 64 tiles, one sequence over K): 4 rows x 256 columns,
// K 1024, 60 us.
#include "common.h"

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

// EPI 0: C = acc (+R).  EPI 1: B is [2N, K] (gate rows then up rows); C = silu(A Bg^T) * (A Bu^T).
// With a GroupedArgs map, row tile blockIdx.y covers rows tile_row0 .. +tile_rows of the expert-sorted order, reads A
// rows through a_gather and uses expert tile_expert's slice of B.
template <int EPI, int MT, int NT, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void gemm_f32_kernel(const F32Gemm p) {
    constexpr int NB = EPI == 1 ? 2 * NT : NT;   // column tiles of B (SwiGLU: gate tiles, then up tiles)
    constexpr int PT = MT > 2 ? 1 : MT;          // row tiles that are added up at a time
    __shared__ floatx4 part[WAVES][PT * NB][64];
    __shared__ float ssq[WAVES][MT * 16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
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
    // lane (r, c) holds k = 16 q + 4 c .. + 3 of row r: MFMA e takes element e of every lane, so a chunk's products are
    // added in the order k = e, 4 + e, 8 + e, 12 + e, the same for both operands
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
    floatx4 acc[MT][NB];
    float ss[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        ss[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int nq = (p.K + F32_CHUNK - 1) / F32_CHUNK;
    constexpr int UN = MT * NB > 4 ? 2 : 4;   // chunks in flight (chunks past K load zeros)
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
    if (p.norm_g) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            ss[i] += __shfl_xor(ss[i], 16, 64);
            ss[i] += __shfl_xor(ss[i], 32, 64);
            if (c == 0) ssq[w][i * 16 + r] = ss[i];
        }
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
    if (!grouped && small_tiles <= 2048) {
        gemm_f32_kernel<EPI, 1, 1, WAVES><<<dim3((p.N + 15) / 16, (unsigned)((p.M + 15) / 16)), WAVES * 64, 0, s>>>(p);
    } else if (!grouped && big_tiles >= 256 && (EPI == 0 || p.K >= 2048)) {
        gemm_f32_kernel<EPI, 4, BN / 16, WAVES><<<dim3((p.N + BN - 1) / BN, (unsigned)((p.M + 63) / 64)), WAVES * 64, 0, s>>>(p);
    } else {
        const unsigned rows = grouped ? (unsigned)p.g.n_mtiles : (unsigned)((p.M + 31) / 32);
        gemm_f32_kernel<EPI, 2, 2, WAVES><<<dim3((p.N + 31) / 32, rows), WAVES * 64, 0, s>>>(p);
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
