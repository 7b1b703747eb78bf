// bf16 MFMA GEMM for the prefill-size projections and the grouped expert
// GEMMs:  C[M, N] = X[M, K] W[N, K]^T, fp32 accumulation, both operands
// contiguous along K.
//
// Shape of the kernel (gfx950):
//  * one workgroup = one 256 x 256 output tile, 8 wavefronts of 128 x 64, K walked
//    in tiles of 64 (a k-tile row is one 128-byte line);
//  * the k-tiles of X and W pass through LDS as half tiles of 128 rows (16 KB), a
//    ring of eight of them (two k-tiles, 128 KB), filled by 16-byte direct-to-LDS
//    global loads; a half tile is requested eight phases before the one that reads
//    it and has six phases (about 3000 clocks) to arrive;
//  * one k-tile = four phases, one per quarter of the wave's output: read the half
//    tile the quarter needs newly (X0, W1, X1, then W0 of the next k-tile; the
//    other operand is still in registers), request one half tile, join a barrier,
//    run 16 MFMAs, join a barrier.  The two wavefronts that share a SIMD belong to
//    different groups that run half a phase apart, so one group's MFMAs (256
//    clocks of the matrix pipe) cover the other group's reads and requests.
//    Barriers wait for LDS reads and for all but the newest 12 loads, so nothing
//    drains.  Matrix pipe busy: 90 % of the clocks (counters; 74 % in the form
//    before, eight wavefronts that read, load and multiply in lock step);
//  * v_mfma_f32_16x16x32_bf16: the chip runs this kernel at its power limit, and
//    this form spends less than 32x32x16 (half the accumulator traffic per flop):
//    1.30 against 1.14 PFLOP/s with the same schedule, same bits;
//  * a half-tile row is 64 bf16 = 8 chunks of 16 bytes, chunk index XOR-ed with
//    (row / 2) % 8: 64 banks of 4 bytes are two rows, and 16 lanes reading 16
//    consecutive rows at one k-offset (an MFMA fragment read, ds_read_b128) touch
//    16 different 16-byte bank groups;
//  * the WEIGHT rows are the MFMA rows and the ACTIVATION rows the MFMA columns, so
//    each lane ends up holding 4 consecutive output columns of one output row: the
//    epilogue stages 32-row slabs in LDS as fp32 and writes 16-byte row-contiguous
//    stores, residual rows requested one slab ahead;
//  * epilogues: 0 = plain / + residual (fp32 add before the bf16 round), 1 =
//    SwiGLU on a stacked gate/up weight (each wave holds the gate and the up
//    tile of the same columns), 2 = fp32 output (router logits); per-row
//    scaling for the routed experts;
//  * workgroup ids are remapped so that each XCD (own L2) gets a contiguous
//    range of tiles, walked in groups of 4 row tiles per column tile (8: the down
//    projection 3 % slower, the others equal; 16: 7 .. 13 % slower).
// Bound: the power limit (90 % matrix-pipe busy at 1.52 GHz; with the loads served
// from L2 the clock rises to 1.66).  8B-shaped layer, 32768 rows, before -> now:
// QKV 1479 -> 1297 us, O 1045 -> 922, gate/up 6290 -> 5560 (1.38 PFLOP/s), down
// 3418 -> 2890 (1.33); 1652 rows 104 -> 92, 91 -> 79, 419 -> 371, 304 -> 253.
#include <type_traits>

#include "common.h"

#define GEMM_BK 64   // k-tile: a row of it is one 128-byte line

struct GemmParams {
    const bf16* X;
    const bf16* W;
    const bf16* R;
    bf16* C;
    int64_t M;
    int N;  // output columns (F for the SwiGLU epilogue, whose W has 2N rows)
    int K;
    int n_mtiles, n_ntiles;
    int r_f32;  // the residual R is fp32 rather than bf16
    GroupedArgs g;
};

// Waits until at most N_IN_FLIGHT of this wave's global loads are outstanding (the older ones have landed in
// LDS) and all of its LDS reads have returned, then joins the workgroup barrier.  Unlike __syncthreads() it
// does not drain the newer loads.
template <int N_IN_FLIGHT>
__device__ __forceinline__ void ring_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(N_IN_FLIGHT >= 0 && N_IN_FLIGHT < 64, "vector-memory counter is 6 bits");
    __builtin_amdgcn_sched_barrier(0);
    // simm16: vmcnt[3:0] | expcnt (7 = no wait) << 4 | lgkmcnt (0) << 8 | vmcnt[5:4] << 14
    __builtin_amdgcn_s_waitcnt((N_IN_FLIGHT & 15) | (7 << 4) | (0 << 8) | ((N_IN_FLIGHT >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}
__device__ __forceinline__ void plain_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}
__device__ __forceinline__ void wave_priority_high() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_setprio(1);
#endif
}
__device__ __forceinline__ void wave_priority_normal() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_setprio(0);
#endif
}

template <int EPI, bool GROUPED>
__global__ __launch_bounds__(512) void gemm_bf16_kernel(const GemmParams p) {
    constexpr int BM = 256, BN = 256, WM = 2, WN = 4, BK = GEMM_BK;
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;   // 128 x 64 per wave, 8 x 4 MFMA tiles
    constexpr int HT = 128 * BK;                    // elements of a half tile (one LDS slot)
    constexpr int OUTN = EPI == 1 ? BN / 2 : BN;
    constexpr int WOUT = EPI == 1 ? WTN / 2 : WTN;  // output columns per wave
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* lds = reinterpret_cast<bf16*>(smem);

    // ---- which tile -------------------------------------------------------
    const int total = gridDim.x;
    const int per = total / 8, rem = total % 8;
    const int xcd = blockIdx.x % 8, loc = blockIdx.x / 8;
    const int pid = xcd * per + min(xcd, rem) + loc;
    constexpr int GM = 4;
    const int per_group = GM * p.n_ntiles;
    const int first_m = (pid / per_group) * GM;
    const int gsize = min(GM, p.n_mtiles - first_m);
    const int tm = first_m + (pid % per_group) % gsize;
    const int tn = (pid % per_group) / gsize;

    int64_t m0;
    int rows_valid;
    const bf16* Wb = p.W;
    if (GROUPED) {
        const int e = p.g.tile_expert[tm];
        if (e < 0) return;
        m0 = p.g.tile_row0[tm];
        rows_valid = p.g.tile_rows[tm];
        Wb += (int64_t)e * p.g.b_expert_stride;
    } else {
        m0 = (int64_t)tm * BM;
        rows_valid = (int)min((int64_t)BM, p.M - m0);
    }
    const int n0 = tn * OUTN;

    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, c4 = lane >> 4;

    // ---- global -> LDS staging (direct-to-LDS 16-byte loads) ---------------------
    // Half tiles q = 0: W0, 1: X0, 2: W1, 3: X1 (the order they are read in).  Half i of X holds tile rows
    // wm * 128 + i * 64 + .., half j of W the columns wn * 64 + j * 32 + .. of every wave (SwiGLU: half 0 the
    // gate rows, half 1 the up rows of the same columns).  One wave instruction fills 1 KB = 8 rows of 8
    // chunks, lane l at (row l / 8, position l % 8); position = chunk ^ ((row / 2) % 8), so the lane fetches
    // chunk (l % 8) ^ ((row / 2) % 8) of its row.  A half tile is two instructions of every wave.
    const bf16* src[4][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row = (wave * 2 + u) * 8 + (lane >> 3);   // row of the half tile
        const int c = (lane & 7) ^ ((row >> 1) & 7);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int trow = min((row >> 6) * 128 + i * 64 + (row & 63), rows_valid - 1);
            int64_t sr = m0 + trow;
            if (GROUPED && p.g.a_gather) sr = p.g.a_gather[sr];
            src[1 + 2 * i][u] = p.X + sr * p.K + c * 8;
            int n;
            if (EPI == 1)
                n = min(n0 + row, p.N - 1) + i * p.N;
            else
                n = min(n0 + (row >> 5) * 64 + i * 32 + (row & 31), p.N - 1);
            src[2 * i][u] = Wb + (int64_t)n * p.K + c * 8;
        }
    }

    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int nk = p.K / BK;
    // LDS element offsets of a fragment: row r of 64 elements, chunk (4 kk + c4) ^ ((r / 2) % 8)
    int foff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) foff[kk] = r * BK + (((4 * kk + c4) ^ ((r >> 1) & 7)) << 3);
    const bf16* xs = lds + wm * 64 * BK;
    const bf16* ws = lds + wn * 32 * BK;

    auto gload = [&](auto qtag, int kt, int buf) {
        constexpr int q = decltype(qtag)::value;
        bf16* dst = lds + (buf * 4 + q) * HT + wave * 2 * 8 * BK;
        const int k0 = kt * BK;
        load16_to_lds(src[q][0] + k0, dst);
        load16_to_lds(src[q][1] + k0, dst + 8 * BK);
    };
    bf16x8 xf[4][2];
    auto read_w = [&](auto jtag, int buf, bf16x8 (&f)[2][2]) {
        constexpr int q = 2 * decltype(jtag)::value;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                f[nt][kk] = *reinterpret_cast<const bf16x8*>(ws + (buf * 4 + q) * HT + nt * 16 * BK + foff[kk]);
    };
    auto read_x = [&](auto itag, int buf) {
        constexpr int q = 1 + 2 * decltype(itag)::value;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                xf[mt][kk] = *reinterpret_cast<const bf16x8*>(xs + (buf * 4 + q) * HT + mt * 16 * BK + foff[kk]);
    };
    auto mfmas = [&](auto itag, auto jtag, const bf16x8 (&wf)[2][2]) {
        constexpr int i = decltype(itag)::value, j = decltype(jtag)::value;
        wave_priority_high();
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            const int kk = n >> 3, mt = (n >> 1) & 3, nt = (n & 1) ^ (mt & 1);
            acc[4 * i + mt][2 * j + nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt][kk], xf[mt][kk], acc[4 * i + mt][2 * j + nt], 0, 0, 0);
        }
        wave_priority_normal();
        plain_barrier();
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 3> I3;

    // One k-tile = four phases (X0 W0, X0 W1, X1 W1, X1 W0); wa holds W0 of this tile, wb receives W1 and then W0
    // of the next.  The loads of k-tile kt + 2 go out one half tile per phase, and 12 of them (six half tiles)
    // may still fly when the next phase's operands must be there.  Past the end of K the last k-tile is loaded
    // again (into slots nobody reads) rather than branching.
    auto k_tile = [&](int kt, int buf, bf16x8 (&wa)[2][2], bf16x8 (&wb)[2][2]) {
        const int kn = min(kt + 2, nk - 1);
        read_x(I0{}, buf);
        gload(I0{}, kn, buf);
        ring_barrier<12>();
        mfmas(I0{}, I0{}, wa);
        read_w(I1{}, buf, wb);
        gload(I1{}, kn, buf);
        ring_barrier<12>();
        mfmas(I0{}, I1{}, wb);
        read_x(I1{}, buf);
        gload(I2{}, kn, buf);
        ring_barrier<12>();
        mfmas(I1{}, I1{}, wb);
        read_w(I0{}, buf ^ 1, wb);
        gload(I3{}, kn, buf);
        ring_barrier<12>();
        mfmas(I1{}, I0{}, wa);
    };

    // prologue: all half tiles of k-tiles 0 and 1; W0 and X0 of k-tile 0 have landed when all but 12 have
    {
        const int k1 = min(1, nk - 1);
        gload(I0{}, 0, 0);
        gload(I1{}, 0, 0);
        gload(I2{}, 0, 0);
        gload(I3{}, 0, 0);
        gload(I0{}, k1, 1);
        gload(I1{}, k1, 1);
        gload(I2{}, k1, 1);
        gload(I3{}, k1, 1);
    }
    bf16x8 wA[2][2], wB[2][2];
    ring_barrier<12>();
    read_w(I0{}, 0, wA);
    ring_barrier<12>();
    if (wm) plain_barrier();   // the second wave group runs half a phase behind the first
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        k_tile(kt, 0, wA, wB);
        k_tile(kt + 1, 1, wB, wA);
    }
    if (kt < nk) k_tile(kt, 0, wA, wB);
    if (!wm) plain_barrier();

    // ---- epilogue: 32 output rows per pass through a wave-private fp32 slab ----
    // acc[i][j][e]: output row m = wm*WTM + i*16 + r, column n = j*16 + c4*4 + e.  A pass's residual rows are
    // requested one pass ahead; the slab needs no workgroup barrier.
    constexpr int SLD = WOUT + 4;
    constexpr int NCH = WOUT / 8;       // 8-column chunks per row
    constexpr int NU = 32 * NCH / 64;   // chunks per lane and pass
    const bool has_r = EPI != 1 && p.R != nullptr;
    floatx4 rv[2][NU][2];
    auto load_r = [&](int i, floatx4 (&v)[NU][2]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int row = (lane + 64 * u) / NCH, c = (lane + 64 * u) % NCH;
            const int lm = wm * WTM + i * 32 + row;
            const int n = n0 + wn * WOUT + c * 8;
            if (lm >= rows_valid || n >= p.N) continue;
            const int64_t o = (m0 + lm) * p.N + n;
            if (p.r_f32) {
                const floatx4* rf = reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(p.R) + o);
                v[u][0] = rf[0];
                v[u][1] = rf[1];
            } else {
                v[u][0] = *reinterpret_cast<const floatx4*>(p.R + o);
            }
        }
    };
    ring_barrier<0>();   // the repeated loads of the last k-tile must not land in the slabs
    if (has_r) load_r(0, rv[0]);
    float* slab = reinterpret_cast<float*>(smem) + wave * 32 * SLD;
#pragma unroll
    for (int i = 0; i < TM / 2; ++i) {
        if (has_r && i + 1 < TM / 2) load_r(i + 1, rv[(i + 1) & 1]);
        constexpr int TJ = EPI == 1 ? TN / 2 : TN;
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                floatx4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float a = acc[2 * i + g][j][e];
                    if (EPI == 1) {
                        const float u = acc[2 * i + g][j + TN / 2][e];
                        a = a / (1.0f + __expf(-a)) * u;
                    }
                    v[e] = a;
                }
                *reinterpret_cast<floatx4*>(slab + (g * 16 + r) * SLD + j * 16 + c4 * 4) = v;
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int row = (lane + 64 * u) / NCH, c = (lane + 64 * u) % NCH;
            const int lm = wm * WTM + i * 32 + row;  // row inside the tile
            const int n = n0 + wn * WOUT + c * 8;
            float v[8];
            const floatx4 a = *reinterpret_cast<const floatx4*>(slab + row * SLD + c * 8);
            const floatx4 b = *reinterpret_cast<const floatx4*>(slab + row * SLD + c * 8 + 4);
            if (lm >= rows_valid || n >= p.N) continue;
            const int64_t gm = m0 + lm;
            v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
            v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
            if (GROUPED && p.g.row_scale) {
                const float sc = p.g.row_scale[gm];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] *= sc;
            }
            if (has_r && p.r_f32) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] += rv[i & 1][u][0][e];
                    v[4 + e] += rv[i & 1][u][1][e];
                }
            } else if (has_r) {
                const bf16x8 rb = __builtin_bit_cast(bf16x8, rv[i & 1][u][0]);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += (float)rb[e];
            }
            if (EPI == 2) {   // fp32 output (router logits)
                float* cf = reinterpret_cast<float*>(p.C) + gm * p.N + n;
                *reinterpret_cast<floatx4*>(cf) = floatx4{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<floatx4*>(cf + 4) = floatx4{v[4], v[5], v[6], v[7]};
            } else {
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
                *reinterpret_cast<bf16x8*>(p.C + gm * p.N + n) = o;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int EPI, bool GROUPED>
static int launch_cfg(compact_ctx* ctx, GemmParams& p, hipStream_t s) {
    constexpr int OUTN = EPI == 1 ? 128 : 256;
    if (!GROUPED) p.n_mtiles = (int)((p.M + 255) / 256);
    p.n_ntiles = (p.N + OUTN - 1) / OUTN;
    constexpr size_t ring_bytes = (size_t)8 * 128 * GEMM_BK * sizeof(bf16);
    constexpr size_t slab_bytes = (size_t)8 * 32 * (OUTN / 4 + 4) * sizeof(float);
    constexpr size_t smem = ring_bytes > slab_bytes ? ring_bytes : slab_bytes;
    auto kern = gemm_bf16_kernel<EPI, GROUPED>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int64_t tiles = (int64_t)p.n_mtiles * p.n_ntiles;
    if (tiles == 0) return COMPACT_OK;
    kern<<<dim3((unsigned)tiles), 512, smem, s>>>(p);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// Row-tile height used for the grouped expert GEMMs.
int gemm_bf16_mtile() { return 256; }

int launch_gemm_bf16(compact_ctx* ctx, const bf16* A, const bf16* B, const void* R, bool r_f32, bf16* C, int64_t M, int N,
                     int K, int epilogue, const GroupedArgs* grouped, hipStream_t s) {
    if (M == 0) return COMPACT_OK;
    if (K % GEMM_BK != 0 || N % 8 != 0) return set_err(ctx, COMPACT_ESHAPE, "bf16 GEMM needs K % 64 == 0 and N % 8 == 0");
    GemmParams p{};
    p.X = A;
    p.W = B;
    p.R = reinterpret_cast<const bf16*>(R);
    p.r_f32 = r_f32 ? 1 : 0;
    p.C = C;
    p.M = M;
    p.N = N;
    p.K = K;
    if (grouped) {
        p.g = *grouped;
        p.n_mtiles = grouped->n_mtiles;
        if (epilogue == 1) return launch_cfg<1, true>(ctx, p, s);
        return launch_cfg<0, true>(ctx, p, s);
    }
    if (epilogue == 1) return launch_cfg<1, false>(ctx, p, s);
    if (epilogue == 2) return launch_cfg<2, false>(ctx, p, s);
    return launch_cfg<0, false>(ctx, p, s);
}
