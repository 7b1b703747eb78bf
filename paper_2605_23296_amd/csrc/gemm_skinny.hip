// Weight-streaming GEMM for the decode step: a handful of activation rows
// (one per block, M <= 64) against a weight matrix that must be read once from
// HBM.  partials[slice][M][N] = X[M, kslice] W[N, kslice]^T in fp32; the
// caller's next row kernel sums the slices in slice order.
//
//  * each wavefront owns 16 weight rows and one K-slice; its 16-byte loads go
//    straight from global memory into the MFMA operand layout (lane (r, c)
//    holds 8 consecutive k of weight row r), all loads of the slice issued
//    before the first MFMA so that a wave keeps 16 KB in flight;
//  * v_mfma_f32_16x16x32_bf16 with the weight rows as MFMA rows and the
//    (zero-padded) activation rows as MFMA columns; the activation slice is
//    staged once per workgroup in LDS;
//  * the K-split depends on K alone, never on the number of activation rows,
//    so a block's result does not depend on the batch it is decoded in.
#include "common.h"
#include "vecio.h"

#define SKINNY_KSLICE 512
#define SKINNY_STEPS (SKINNY_KSLICE / 32)

int skinny_ksplit(int M, int N, int K) {
    (void)M;
    (void)N;
    return (K + SKINNY_KSLICE - 1) / SKINNY_KSLICE;
}

// GROUPED: the grid is flat, blockIdx.x = k-slice, 64 weight rows and expert (slice_item);
// an expert's rows are rows offsets[e] .. offsets[e+1]-1
// of the expert-sorted order (at most MT*16 of them), read from X through
// a_gather (null: X is already in sorted order), multiplied with that expert's
// weight matrix, and the partials keep the sorted order: P[slice][sorted row][N].
// Experts nobody was routed to leave at once.  With a tile map (expert_list =
// the map's experts, tile_row0 / tile_rows its row ranges, tiles of at most MT*16
// rows) it is a tile in the expert's place: an expert with more rows than a tile
// holds is streamed once per tile.
struct SkinnyGroup {
    const int32_t* expert_list;  // [n_tiles] experts to run, -1 = none (null: tile e = expert e)
    const int32_t* tile_row0;    // [n_tiles] first sorted row of the tile (null: the expert's first row)
    const int32_t* tile_rows;    // [n_tiles] rows of the tile (null: all of the expert's rows)
    const int32_t* offsets;   // [E + 1]
    const int32_t* a_gather;  // [total_rows] or null
    int64_t w_expert_stride;  // elements
    int total_rows;
    int n_tiles;              // entries of the list, or experts
};

// Front half of an RMSNorm folded into the activation staging (null g: off): the
// staged operand is bf16(x * g) and the workgroups of the first column tile leave
// ssq_parts[slice][row] = sum of x^2 over the slice; the consumer of the partials
// multiplies by 1 / rms.
// Back half of one (null m_out: off): X holds x * g, the staged operand is bf16(X / rms) with 1 / rms from the column-group
// sums in `rn`, and the workgroups of the first column tile leave it in m_out as well.
struct SkinnyNormIn {
    const bf16* g = nullptr;
    float* ssq_parts = nullptr;
    RowNorm rn;
    bf16* m_out = nullptr;
};

// RING < SKINNY_STEPS: only the first RING loads of the slice go out at once, the rest one per k-step as the
// registers come free (half the registers per wavefront, twice the wavefronts per CU for the same bytes in flight).
template <int MT, bool GROUPED, int WAVES, int RING = SKINNY_STEPS>
__global__ __launch_bounds__(WAVES * 64, RING < SKINNY_STEPS ? 2 : 1) void gemm_skinny_kernel(const bf16* __restrict__ X, const bf16* __restrict__ W,
                                                          float* __restrict__ P, int M, int N, int K, const SkinnyGroup grp,
                                                          const SkinnyNormIn nin) {
    constexpr int LDX = SKINNY_KSLICE + 8;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* xs = reinterpret_cast<bf16*>(smem);  // [MT*16][LDX]
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    int row_base = 0, p_rows = M, slice = blockIdx.x, col = blockIdx.y;
    if (GROUPED) {
        const SliceItem it = slice_item(blockIdx.x, (K + SKINNY_KSLICE - 1) / SKINNY_KSLICE, (N + WAVES * 16 - 1) / (WAVES * 16));
        slice = it.slice;
        col = it.col;
        if (it.tile >= grp.n_tiles) return;
        const int e = grp.expert_list ? grp.expert_list[it.tile] : it.tile;
        if (e < 0) return;
        row_base = grp.tile_row0 ? grp.tile_row0[it.tile] : grp.offsets[e];
        M = min(grp.tile_rows ? grp.tile_rows[it.tile] : grp.offsets[e + 1] - row_base, MT * 16);
        if (M <= 0) return;
        W += (size_t)e * grp.w_expert_stride;
        p_rows = grp.total_rows;
    }
    // the K-slices of the same weight rows are neighbours in the grid: workgroups that
    // run together read whole DRAM pages, not the same slice of far-apart rows.  Grouped
    // (a launch is many rounds of workgroups), they also run on one XCD, where some layers
    // gain and others stay (1 % either way): whole steps of 16 rows, slices in turn to the
    // XCDs -> together: d 2880, F 2880, 128 experts 479 -> 466 us; d 2048, F 1024, 16 experts
    // 79 -> 76; d 2048, F 2048 297 -> 288; d 4096, 2112 and 1600 as before.
    // Four neighbouring lanes on 64 bytes of a row, moved to operand order by cross-lane
    // reads, gained another 1-2 % there and lost 1-4 % where the experts fit the caches.
    const int k0 = slice * SKINNY_KSLICE;
    const int klen = min(SKINNY_KSLICE, K - k0);
    const int nsteps = klen / 32;
    const int r = lane & 15, c = lane >> 4;
    const int n0 = (col * WAVES + wave) * 16;
    const bool active = n0 < N;

    // the weight stream goes first: everything below overlaps with it
    bf16x8 a[RING];
    const bf16* wp = W + (size_t)(min(n0, N - 16) + r) * K + k0 + c * 8;
    if (active) {
#pragma unroll
        for (int s = 0; s < RING; ++s)
            if (s < nsteps) a[s] = *reinterpret_cast<const bf16x8*>(wp + s * 32);
    }

    const int cpr = klen / 8;  // 16-byte chunks per row (at most 64)
    if (!GROUPED && nin.g) {
        // RMSNorm front half: a wavefront stages whole rows, so that the row's sum of
        // squares over this slice is one butterfly (fixed order)
        for (int row = wave; row < M; row += WAVES) {
            bf16x8 v;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (bf16)0.f;
            float ss = 0.f;
            if (lane < cpr) {
                v = *reinterpret_cast<const bf16x8*>(X + (size_t)row * K + k0 + lane * 8);
                const bf16x8 gv = *reinterpret_cast<const bf16x8*>(nin.g + k0 + lane * 8);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float f = (float)v[j];
                    ss += f * f;
                    v[j] = (bf16)(f * (float)gv[j]);
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
            if (lane == 0 && blockIdx.y == 0) nin.ssq_parts[(size_t)slice * M + row] = ss;
            if (lane < cpr) *reinterpret_cast<bf16x8*>(xs + row * LDX + lane * 8) = v;
        }
    } else if (!GROUPED && MT == 1 && nin.m_out) {
        constexpr int RW = 16 / WAVES, PMAX = 8;   // rows per wavefront; parts per lane (nparts <= 512)
        float pv[RW][PMAX];
        bf16x8 v[RW];
        // all loads before the first sum, none of them conditional (past the end: a piece that is dropped)
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int row = min(wave + i * WAVES, M - 1);
            v[i] = *reinterpret_cast<const bf16x8*>(X + (size_t)row * K + k0 + min(lane, cpr - 1) * 8);
#pragma unroll
            for (int u = 0; u < PMAX; ++u) pv[i][u] = nin.rn.ssq_parts[(size_t)min(lane + 64 * u, nin.rn.nparts - 1) * M + row];
        }
        float ss[RW];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int row = wave + i * WAVES;
            ss[i] = 0.f;
#pragma unroll
            for (int u = 0; u < PMAX; ++u) ss[i] += lane + 64 * u < nin.rn.nparts ? pv[i][u] : 0.f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) ss[i] += __shfl_xor(ss[i], o, 64);
            const float rs = 1.0f / sqrtf(ss[i] * nin.rn.inv_d + nin.rn.eps);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[i][j] = row < M ? (bf16)((float)v[i][j] * rs) : (bf16)0.f;
            if (lane < cpr) {
                *reinterpret_cast<bf16x8*>(xs + row * LDX + lane * 8) = v[i];
                if (blockIdx.y == 0 && row < M) *reinterpret_cast<bf16x8*>(nin.m_out + (size_t)row * K + k0 + lane * 8) = v[i];
            }
        }
    } else {
        for (int q = t; q < M * cpr; q += WAVES * 64) {
            const int row = q / cpr, cc = q - row * cpr;
            size_t src = row_base + row;
            if (GROUPED && grp.a_gather) src = grp.a_gather[src];
            const bf16x8 v = *reinterpret_cast<const bf16x8*>(X + src * K + k0 + cc * 8);
            *reinterpret_cast<bf16x8*>(xs + row * LDX + cc * 8) = v;
        }
    }
    __syncthreads();
    if (!active) return;

    floatx4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SKINNY_STEPS; ++s) {
        if (s < nsteps) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x8 b = *reinterpret_cast<const bf16x8*>(xs + min(mt * 16 + r, M - 1) * LDX + s * 32 + c * 8);
                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s % RING], b, acc[mt], 0, 0, 0);
            }
            if (RING < SKINNY_STEPS && s + RING < SKINNY_STEPS && s + RING < nsteps)
                a[s % RING] = *reinterpret_cast<const bf16x8*>(wp + (s + RING) * 32);
        }
    }
    // acc[mt][e]: activation row m = mt*16 + r, weight row n = n0 + 4c + e
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = mt * 16 + r;
        if (m < M) *reinterpret_cast<floatx4*>(P + ((size_t)slice * p_rows + row_base + m) * N + n0 + 4 * c) = acc[mt];
    }
}

template <int MT, int WAVES, int RING = SKINNY_STEPS>
static int launch_skinny_cfg(compact_ctx* ctx, const bf16* A, const bf16* B, float* partials, int M, int N, int K, int ks,
                             const SkinnyNormIn& nin, hipStream_t s) {
    const size_t smem = (size_t)MT * 16 * (SKINNY_KSLICE + 8) * sizeof(bf16);
    static bool attr = false;
    if (!attr && smem > 48 * 1024) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_skinny_kernel<MT, false, WAVES, RING>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr = true;
    }
    dim3 grid(ks, (N + 16 * WAVES - 1) / (16 * WAVES));
    gemm_skinny_kernel<MT, false, WAVES, RING><<<grid, WAVES * 64, smem, s>>>(A, B, partials, M, N, K, SkinnyGroup{}, nin);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// One workgroup = 4 wavefronts (64 weight rows) for up to 16 activation rows; with
// more rows the staged activation slice grows, so 8 wavefronts (128 weight rows)
// share it: half the activation traffic per weight byte, the same number of
// wavefronts per compute unit.
int launch_gemm_skinny(compact_ctx* ctx, const bf16* A, const bf16* B, float* partials, int M, int N, int K, int ks,
                       hipStream_t s, const bf16* norm_g, float* norm_ssq_parts) {
    if (M < 1 || M > 64) return set_err(ctx, COMPACT_ESHAPE, "weight-streaming GEMM takes 1..64 activation rows");
    if (N % 16 != 0 || K % 64 != 0) return set_err(ctx, COMPACT_ESHAPE, "weight-streaming GEMM needs N % 16 == 0 and K % 64 == 0");
    if (ks != skinny_ksplit(M, N, K)) return set_err(ctx, COMPACT_EINVAL, "unexpected K split");
    SkinnyNormIn nin;
    if (norm_g) {
        if (!norm_ssq_parts) return set_err(ctx, COMPACT_EINVAL, "no room for the row sums of squares");
        nin.g = norm_g;
        nin.ssq_parts = norm_ssq_parts;
    }
    // 49 .. 64 rows: two workgroups of 8 wavefronts fit a CU (the staged slice is 66 KB); a grid beyond what the
    // chip holds at once (the q/k/v projection of a layer with d_model 8192: 16 slices x 80 column groups) goes to
    // workgroups of 16 wavefronts with 6 of the 16 loads up front instead: again two per CU, half the activation staging.
    // 64 rows, N 10240, K 8192: 62.9 -> 51.1 us, a whole step of such a layer 181.5 -> 174.4 (at 32 rows the same change
    // cost 2 us and is not made)
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    const bool fat = (int64_t)ks * ((N + 127) / 128) > 2 * (int64_t)n_cus;
    switch ((M + 15) / 16) {
        case 1: return launch_skinny_cfg<1, 4>(ctx, A, B, partials, M, N, K, ks, nin, s);
        case 2: return launch_skinny_cfg<2, 8>(ctx, A, B, partials, M, N, K, ks, nin, s);
        case 3: return launch_skinny_cfg<3, 8>(ctx, A, B, partials, M, N, K, ks, nin, s);
        default: return fat ? launch_skinny_cfg<4, 16, 6>(ctx, A, B, partials, M, N, K, ks, nin, s)
                            : launch_skinny_cfg<4, 8>(ctx, A, B, partials, M, N, K, ks, nin, s);
    }
}

// partials of m B^T for at most 16 rows, m = bf16(hg / rms) left in m_out: the end of an RMSNorm rides in the projection
// that consumes it
int launch_gemm_skinny_rownorm(compact_ctx* ctx, const bf16* hg, const RowNorm& norm, bf16* m_out, const bf16* B, float* partials,
                               int M, int N, int K, int ks, hipStream_t s) {
    if (M < 1 || M > 16 || N % 16 != 0 || K % 64 != 0 || norm.nparts > 512)
        return set_err(ctx, COMPACT_ESHAPE, "folding the end of an RMSNorm into the weight-streaming GEMM needs at most 16 rows");
    if (ks != skinny_ksplit(M, N, K)) return set_err(ctx, COMPACT_EINVAL, "unexpected K split");
    SkinnyNormIn nin;
    nin.rn = norm;
    nin.m_out = m_out;
    return launch_skinny_cfg<1, 4>(ctx, hg, B, partials, M, N, K, ks, nin, s);
}

// Per-expert weight streaming for routed decode rows (at most 16 rows per expert):
// partials[ks][total_rows][N], rows in expert-sorted order.
int launch_gemm_skinny_grouped(compact_ctx* ctx, const bf16* X, const int32_t* a_gather, const bf16* W, int64_t w_expert_stride,
                               const int32_t* offsets, int n_experts, int total_rows, float* partials, int N, int K, int ks,
                               hipStream_t s, const int32_t* expert_list, int n_listed, const int32_t* tile_row0,
                               const int32_t* tile_rows) {
    if (N % 16 != 0 || K % 64 != 0) return set_err(ctx, COMPACT_ESHAPE, "weight-streaming GEMM needs N % 16 == 0 and K % 64 == 0");
    if (ks != skinny_ksplit(1, N, K)) return set_err(ctx, COMPACT_EINVAL, "unexpected K split");
    SkinnyGroup g{expert_list, tile_row0, tile_rows, offsets, a_gather, w_expert_stride, total_rows, expert_list ? n_listed : n_experts};
    const int64_t grid = slice_items(ks, (N + 63) / 64, g.n_tiles);
    if (grid >= 1 << 24) return set_err(ctx, COMPACT_ESHAPE, "too many workgroups for weight streaming");
    const size_t smem = (size_t)16 * (SKINNY_KSLICE + 8) * sizeof(bf16);
    gemm_skinny_kernel<1, true, 4><<<(unsigned)grid, 256, smem, s>>>(X, W, partials, 0, N, K, g, SkinnyNormIn{});
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// C = sum_s partials[s] (+R), rounded to bf16
__global__ __launch_bounds__(256) void skinny_finish_kernel(const float* __restrict__ P, int ks, const bf16* __restrict__ R,
                                                            bf16* __restrict__ C, int M, int N) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t total = (size_t)M * N;
    if (i >= total) return;
    float v = R ? (float)R[i] : 0.f;
    for (int s = 0; s < ks; ++s) v += P[s * total + i];
    C[i] = (bf16)v;
}

int launch_skinny_finish(compact_ctx* ctx, const float* partials, int ks, const bf16* R, bf16* C, int M, int N,
                         hipStream_t s) {
    const size_t total = (size_t)M * N;
    skinny_finish_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>(partials, ks, R, C, M, N);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
