// bf16 MFMA GEMM for the prefill-size projections and the grouped expert
// GEMMs:  C[M, N] = X[M, K] W[N, K]^T, fp32 accumulation, both operands
// contiguous along K.
//
// Shape of the kernel (gfx950):
//  * one workgroup = one 256 x 256 output tile (or a half of one, see tile_128; both
//    kinds share a launch), 8 wavefronts of 128 x 64, K walked in tiles of 64 (a
//    k-tile row is one 128-byte line);
//  * the k-tiles of X and W pass through LDS as half tiles of 128 rows (16 KB), a
//    ring of eight of them (two k-tiles, 128 KB), filled by 16-byte direct-to-LDS
//    global loads; a half tile is requested seven phases before the one that reads
//    it and has six phases (about 3000 clocks) to arrive;
//  * one k-tile = four phases, one per quarter of the wave's output: read the half
//    tile the quarter needs newly (X0, W1, X1, then W0 of the next k-tile; the
//    other operand is still in registers), request one half tile, join a barrier,
//    run 16 MFMAs, join a barrier.  The two wavefronts that share a SIMD belong to
//    different groups that run half a phase apart, so one group's MFMAs (256
//    clocks of the matrix pipe) cover the other group's reads and requests.
//    Barriers wait for LDS reads and for all but the newest 12 loads, so nothing
//    drains.  Matrix pipe busy: 85 to 88 % of the clocks in the 8 x 4096 pass (counters;
//    73 to 75 % in the form before, eight wavefronts that read, load and multiply in
//    lock step);
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
//    tile of the same columns), 2 = fp32 output (router logits, decode partials), 3 =
//    1 with a factor per row (decode); per-row
//    scaling for the routed experts;
//  * workgroup ids are remapped so that each XCD (own L2) gets a contiguous
//    range of tiles, walked in groups of 4 row tiles per column tile (8: the down
//    projection 3 % slower, the others equal; 16: 7 .. 13 % slower).
// Bound: the power limit (the gate/up projection of that pass: matrix pipe 85 % busy at
// 1.60 GHz; a probe whose loads all hit L2 ran at a clock 9 % higher).  8B-shaped layer, 32768
// rows: QKV 1.14 ms, O 0.82, gate/up 5.11 (1.51 PFLOP/s), down 2.52 (1.53); in the form of lock steps 1.48, 1.05, 6.29
// and 3.42.  1652 rows, where rounds of workgroups count: 86, 60, 286 and 195 us (104, 91, 419, 304).
#include <algorithm>
#include <cmath>
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
    int touch;   // 256 x 256 kernel, plain product in halves: weight lines are touched ahead
    int n_full;  // 256 x 256 kernel, plain product: workgroups that take a whole tile (the others take halves)
    int r_f32;  // the residual R is fp32 rather than bf16
    const float* pre_scale;   // epilogue 3: factor of every row's products before the silu (null = 1)
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

// Where a workgroup's tile lies.  Workgroup ids are dealt to the XCDs round robin: each XCD takes a contiguous
// range of tiles, walked in groups of GM row tiles per column tile.
struct TilePos {
    int64_t m0;       // first row
    int rows_valid;   // 0: nothing to do
    int n0;           // first output column
    const bf16* W;    // the weight matrix (the expert's)
};
// workgroup i of n that are dealt round robin -> its place in the order of tiles
__device__ __forceinline__ int xcd_order(int i, int n) {
    const int per = n / 8, rem = n % 8, xcd = i % 8;
    return xcd * per + min(xcd, rem) + i / 8;
}
// place in the order -> row tile, column tile (n_mtiles row tiles)
template <int GM>
__device__ __forceinline__ void tile_at(int pid, int n_mtiles, int n_ntiles, int& tm, int& tn) {
    const int per_group = GM * n_ntiles;
    const int first_m = (pid / per_group) * GM;
    const int gsize = min(GM, n_mtiles - first_m);
    tm = first_m + (pid % per_group) % gsize;
    tn = (pid % per_group) / gsize;
}
template <bool GROUPED, int BM, int OUTN, int GM>
__device__ __forceinline__ TilePos find_tile(const GemmParams& p) {
    int tm, tn;
    tile_at<GM>(xcd_order(blockIdx.x, gridDim.x), p.n_mtiles, p.n_ntiles, tm, tn);
    TilePos tp;
    tp.n0 = tn * OUTN;
    tp.W = p.W;
    if (GROUPED) {
        const int e = p.g.tile_expert[tm];
        tp.m0 = e < 0 ? 0 : p.g.tile_row0[tm];
        tp.rows_valid = e < 0 ? 0 : p.g.tile_rows[tm];
        tp.W += (int64_t)max(e, 0) * p.g.b_expert_stride;
    } else {
        tp.m0 = (int64_t)tm * BM;
        tp.rows_valid = (int)min((int64_t)BM, p.M - tp.m0);
    }
    return tp;
}

// Epilogue of one wavefront: TM x TN MFMA tiles, 32 output rows per pass through a wave-private fp32 slab
// [32][WOUT + 4].  acc[i][j][e]: output row wrow + i*16 + r of the tile, column n_first + j*16 + c4*4 + e (SwiGLU: the
// first TN / 2 tiles are the gate, the others the up values of the same columns).  A pass's residual rows are
// requested one pass ahead; the slab needs no workgroup barrier.
template <int EPI, bool GROUPED, int TM, int TN>
__device__ __forceinline__ void store_tile(const GemmParams& p, const floatx4 (&acc)[TM][TN], float* slab, int lane, int wrow,
                                           int rows_valid, int64_t m0, int n_first) {
    constexpr bool GLU = EPI == 1 || EPI == 3;
    constexpr int WOUT = (GLU ? TN / 2 : TN) * 16;
    constexpr int SLD = WOUT + 4;
    constexpr int NCH = WOUT / 8;       // 8-column chunks per row
    constexpr int NU = 32 * NCH / 64;   // chunks per lane and pass
    static_assert(TM % 2 == 0 && NU >= 1, "passes of 32 rows, at least one chunk per lane");
    const int r = lane & 15, c4 = lane >> 4;
    const bool has_r = !GLU && p.R != nullptr;
    floatx4 rv[2][NU][2];
    auto load_r = [&](int i, floatx4 (&v)[NU][2]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int row = (lane + 64 * u) / NCH, c = (lane + 64 * u) % NCH;
            const int lm = wrow + i * 32 + row, n = n_first + c * 8;
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
    if (has_r) load_r(0, rv[0]);
#pragma unroll
    for (int i = 0; i < TM / 2; ++i) {
        if (has_r && i + 1 < TM / 2) load_r(i + 1, rv[(i + 1) & 1]);
        constexpr int TJ = GLU ? TN / 2 : TN;
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                floatx4 v;
                const float ps = EPI == 3 && p.pre_scale ? p.pre_scale[m0 + min(wrow + i * 32 + g * 16 + r, rows_valid - 1)] : 1.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float a = acc[2 * i + g][j][e];
                    if (GLU) {
                        float u = acc[2 * i + g][j + TN / 2][e];
                        if (EPI == 3) {
                            a *= ps;
                            u *= ps;
                        }
                        // A division to half a unit in the last place is ten instructions, 64 times a lane, while the matrix
                        // pipe waits.  The reciprocal instruction (one and a half units with its product) saves 1 to 2 % (2 * 14336
                        // x 4096 at 32768 rows 5111 -> 5069 us, routed 16 x 8192 13874 -> 13581), but changes a bf16
                        // result in one of 180000 places.
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
            const int lm = wrow + i * 32 + row, n = n_first + c * 8;
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
__device__ __forceinline__ void tile_256(const GemmParams& p, const TilePos& tp, char* smem) {
    constexpr int BM = 256, BN = 256, WM = 2, WN = 4, BK = GEMM_BK;
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;   // 128 x 64 per wave, 8 x 4 MFMA tiles
    constexpr int HT = 128 * BK;                    // elements of a half tile (one LDS slot)
    constexpr int WOUT = EPI == 1 ? WTN / 2 : WTN;  // output columns per wave
    bf16* lds = reinterpret_cast<bf16*>(smem);
    const int64_t m0 = tp.m0;
    const int rows_valid = tp.rows_valid, n0 = tp.n0;
    const bf16* Wb = tp.W;

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

    ring_barrier<0>();   // the repeated loads of the last k-tile must not land in the slabs
    store_tile<EPI, GROUPED, TM, TN>(p, acc, reinterpret_cast<float*>(smem) + wave * 32 * (WOUT + 4), lane, wm * WTM, rows_valid, m0,
                                     n0 + wn * WOUT);
}

// ---------------------------------------------------------------------------
// The same schedule over 128 x 256 tiles (wavefronts of 64 x 64, two phases per k-tile: X0 W0, X0 W1): twice the
// workgroups for calls whose 256 x 256 tiles would leave half the chip idle.  A k-tile is three half tiles (W0, X0,
// W1); the ring holds three k-tiles (nine slots, 144 KB).  A phase requests three of the six 8-row pieces a wavefront
// owns of a k-tile; 11 or 12 of them may still fly when the next phase's operands must be there.
// ---------------------------------------------------------------------------
// TOUCH: weight lines are touched ahead of the ring, this workgroup's share among eight of the same columns.  A CU has some 50
// KB of loads in flight, so weights that come from HBM, 900 ns away, limit it to 27 bytes a clock, a k-tile to 0.85 us, whatever
// the ring holds; all eight workgroups ask for the same lines at the same time and wait alike.  With an eighth of the lines
// touched by each of them four k-tiles ahead, the loads find them in the L2 (eight k-tiles ahead 1 % slower, sixteen 3 %; with
// four sharers at 700 rows 48 -> 50 us).  Row tiles behind the last whole group of four and a bottom half tile touch nothing (80
// of 208 workgroups at 1652 rows and N 4096), and where the XCDs' ranges of the order cut a group of sharers in two (3 of the 16
// groups there), either L2 holds only the lines that its own workgroups touched.
template <int EPI, bool GROUPED, bool TOUCH>
__device__ __forceinline__ void tile_128(const GemmParams& p, const TilePos& tp, char* smem, int share) {
    constexpr int WN = 4, BK = GEMM_BK;
    constexpr int WTM = 64, WTN = 64, TM = WTM / 16, TN = WTN / 16;
    constexpr int HT = 128 * BK;
    constexpr int WOUT = EPI == 1 ? WTN / 2 : WTN;
    bf16* lds = reinterpret_cast<bf16*>(smem);
    const int n0 = tp.n0;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, c4 = lane >> 4;

    // half tiles q = 0: W0, 1: X0, 2: W1 (the order they are read in); pieces, chunks and swizzle as above
    const bf16* src[3][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row = (wave * 2 + u) * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        int64_t sr = tp.m0 + min(row, tp.rows_valid - 1);
        if (GROUPED && p.g.a_gather) sr = p.g.a_gather[sr];
        src[1][u] = p.X + sr * p.K + c * 8;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            int n;
            if (EPI == 1)
                n = min(n0 + row, p.N - 1) + j * p.N;
            else
                n = min(n0 + (row >> 5) * 64 + j * 32 + (row & 31), p.N - 1);
            src[2 * j][u] = tp.W + (int64_t)n * p.K + c * 8;
        }
    }
    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int nk = p.K / BK;
    int foff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) foff[kk] = r * BK + (((4 * kk + c4) ^ ((r >> 1) & 7)) << 3);
    const bf16* xs = lds + wm * 64 * BK;
    const bf16* ws = lds + wn * 32 * BK;
    // piece u of half tile q of k-tile kt, into k-tile buffer buf
    auto gload = [&](int q, int u, int kt, int buf) {
        load16_to_lds(src[q][u] + min(kt, nk - 1) * BK, lds + (buf * 3 + q) * HT + (wave * 2 + u) * 8 * BK);
    };
    auto read_w = [&](int j, int buf, bf16x8 (&f)[2][2]) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
                f[nt][kk] = *reinterpret_cast<const bf16x8*>(ws + (buf * 3 + 2 * j) * HT + nt * 16 * BK + foff[kk]);
    };
    // wavefront `share` touches a line of each of 64 of the tile's weight rows, of every other k-tile
    const bf16* tsrc = nullptr;
    if (TOUCH) {
        const int row = (wave & 3) * 64 + lane;
        const int n = EPI == 1 ? min(n0 + (row & 127), p.N - 1) + (row >> 7) * p.N : min(n0 + row, p.N - 1);
        tsrc = tp.W + (int64_t)n * p.K;
    }
    auto touch = [&](int kt) __attribute__((always_inline)) {
        if (TOUCH && wave == share && (kt & 1) == wave >> 2 && kt < nk)
            load4_to_lds(tsrc + kt * BK, smem + 9 * HT * sizeof(bf16) + wave * 256);
    };
    bf16x8 xf[4][2], w0[2][2], w1[2][2];
    auto mfmas = [&](auto jtag, const bf16x8 (&wf)[2][2]) {
        constexpr int j = decltype(jtag)::value;
        wave_priority_high();
#pragma unroll
        for (int n = 0; n < 16; ++n) {
            const int kk = n >> 3, mt = (n >> 1) & 3, nt = (n & 1) ^ (mt & 1);
            acc[mt][2 * j + nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[nt][kk], xf[mt][kk], acc[mt][2 * j + nt], 0, 0, 0);
        }
        wave_priority_normal();
        plain_barrier();
    };
    // k-tile kt in buffer b0, kt + 1 in b1, kt + 2 in b2
    auto k_tile = [&](int kt, int b0, int b1, int b2) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                xf[mt][kk] = *reinterpret_cast<const bf16x8*>(xs + (b0 * 3 + 1) * HT + mt * 16 * BK + foff[kk]);
        gload(2, 0, kt + 2, b2);
        gload(2, 1, kt + 2, b2);
        gload(0, 0, kt + 3, b0);
        touch(kt + 4);
        ring_barrier<11>();
        mfmas(std::integral_constant<int, 0>{}, w0);
        read_w(1, b0, w1);
        read_w(0, b1, w0);
        gload(0, 1, kt + 3, b0);
        gload(1, 0, kt + 3, b0);
        gload(1, 1, kt + 3, b0);
        ring_barrier<12>();
        mfmas(std::integral_constant<int, 1>{}, w1);
    };
    // prologue: k-tiles 0 and 1, and W0, X0 of k-tile 2; the first two half tiles have landed when all but 12 pieces have
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int q = 0; q < (i == 2 ? 2 : 3); ++q) {
            gload(q, 0, i, i);
            gload(q, 1, i, i);
        }
    ring_barrier<12>();
    read_w(0, 0, w0);
    ring_barrier<12>();
    if (wm) plain_barrier();   // the second wave group runs half a phase behind the first
    int kt = 0;
    for (; kt + 2 < nk; kt += 3) {
        k_tile(kt, 0, 1, 2);
        k_tile(kt + 1, 1, 2, 0);
        k_tile(kt + 2, 2, 0, 1);
    }
    if (kt < nk) k_tile(kt, 0, 1, 2);
    if (kt + 1 < nk) k_tile(kt + 1, 1, 2, 0);
    if (!wm) plain_barrier();
    ring_barrier<0>();   // the repeated loads of the last k-tile must not land in the slabs
    store_tile<EPI, GROUPED, TM, TN>(p, acc, reinterpret_cast<float*>(smem) + wave * 32 * (WOUT + 4), lane, wm * WTM, tp.rows_valid,
                                     tp.m0, n0 + wn * WOUT);
}

// Plain products: the output is cut into slots of 256 x 256 (groups of 4 row tiles, as above); the first n_full of them
// are a workgroup each, the others two workgroups of 128 x 256, and last come the halves of a bottom row tile of at most
// 128 rows: a last round that whole tiles would fill by half or less takes half tiles, which need 0.6 of the time, and the
// short ones fill units that the round leaves idle.  Against one form for all of a call (us): 2 * 14336 x 4096 at 1652 rows
// 351 -> 280 (672 whole and 112 half tiles; before, 1456 halves), N 4096 K 14336 at 4600 rows 478 -> 446, at 9000 rows
// 877 -> 774, N 5120 K 2880 at 4600 rows 106 -> 95; the other calls of a sweep of 8 products at 40 row counts within 1 %.
// Routed products: a workgroup per tile of the map, in the form that its rows need.
template <int EPI, bool GROUPED>
__global__ __launch_bounds__(512) void gemm_bf16_kernel(const GemmParams p) {
    constexpr int OUTN = EPI == 1 ? 128 : 256;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    if constexpr (GROUPED) {
        const TilePos tp = p.g.mtile == 256 ? find_tile<true, 256, OUTN, 4>(p) : find_tile<true, 128, OUTN, 8>(p);
        if (tp.rows_valid <= 0) return;
        if (tp.rows_valid > 128)
            tile_256<EPI, true>(p, tp, smem);
        else
            tile_128<EPI, true, false>(p, tp, smem, 0);
    } else {
        const int i = blockIdx.x;
        int tm, tn;
        TilePos tp;
        tp.W = p.W;
        if (i < p.n_full) {
            tile_at<4>(xcd_order(i, p.n_full), p.n_mtiles, p.n_ntiles, tm, tn);
            tp.m0 = (int64_t)tm * 256;
            tp.n0 = tn * OUTN;
            tp.rows_valid = (int)min((int64_t)256, p.M - tp.m0);
            tile_256<EPI, false>(p, tp, smem);
        } else {
            const int h = xcd_order(i - p.n_full, gridDim.x - p.n_full);
            const int slot = p.n_full + h / 2, slots = p.n_mtiles * p.n_ntiles;
            int share = -1;
            if (slot < slots) {
                tile_at<4>(slot, p.n_mtiles, p.n_ntiles, tm, tn);
                tp.m0 = (int64_t)tm * 256 + (h & 1) * 128;
                if (p.touch && tm / 4 * 4 + 4 <= p.n_mtiles) share = tm % 4 * 2 + (h & 1);
            } else {
                tn = h - 2 * (slots - p.n_full);
                tp.m0 = (int64_t)p.n_mtiles * 256;
            }
            tp.n0 = tn * OUTN;
            tp.rows_valid = (int)min((int64_t)128, p.M - tp.m0);
            if (share >= 0)
                tile_128<EPI, false, true>(p, tp, smem, share);
            else
                tile_128<EPI, false, false>(p, tp, smem, 0);
        }
    }
}

// ---------------------------------------------------------------------------
// Smaller tiles, for calls whose 256 x 256 tiles would leave compute units idle: BM x BN outputs per workgroup of
// WM x WN wavefronts, k-tiles of 64 in a ring of S LDS stages, one barrier per k-tile, S - 1 k-tiles of loads in
// flight.  Same layout, same MFMAs in the same order along K as above: an output has the same bits whichever tile it
// lies in.
// ---------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, int S, int EPI, bool GROUPED>
__global__ __launch_bounds__(WM* WN * 64) void gemm_bf16_small_kernel(const GemmParams p) {
    constexpr bool GLU = EPI == 1 || EPI == 3;
    constexpr int NW = WM * WN, BK = GEMM_BK;
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
    constexpr int STAGE = (BM + BN) * BK;   // elements
    constexpr int OUTN = GLU ? BN / 2 : BN;
    constexpr int WOUT = GLU ? WTN / 2 : WTN;
    constexpr int XU = BM / 8 / NW, WU = BN / 8 / NW;   // 8-row load units per wavefront
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && TN % 2 == 0, "tile rows must split over the wavefronts");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* lds = reinterpret_cast<bf16*>(smem);
    const TilePos tp = find_tile<GROUPED, BM, OUTN, 8>(p);
    if (tp.rows_valid <= 0) return;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, c4 = lane >> 4;

    const bf16 *xsrc[XU], *wsrc[WU];
#pragma unroll
    for (int u = 0; u < XU; ++u) {
        const int row = (wave * XU + u) * 8 + (lane >> 3);
        int64_t sr = tp.m0 + min(row, tp.rows_valid - 1);
        if (GROUPED && p.g.a_gather) sr = p.g.a_gather[sr];
        xsrc[u] = p.X + sr * p.K + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    }
#pragma unroll
    for (int u = 0; u < WU; ++u) {
        const int row = (wave * WU + u) * 8 + (lane >> 3);
        int n;
        if (GLU)
            n = row < BN / 2 ? min(tp.n0 + row, p.N - 1) : p.N + min(tp.n0 + row - BN / 2, p.N - 1);
        else
            n = min(tp.n0 + row, p.N - 1);
        wsrc[u] = tp.W + (int64_t)n * p.K + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    }
    // gridDim.y slices of K (partial results, slice by slice in C): this workgroup's k-tiles
    const int k_lo = p.K / BK * blockIdx.y / gridDim.y, nk = p.K / BK * (blockIdx.y + 1) / gridDim.y - k_lo;
    auto gload = [&](int kt, int stage) {
        const int k0 = (k_lo + min(kt, nk - 1)) * BK;   // past the end: the last k-tile again, into a stage nobody reads
        bf16* dst = lds + stage * STAGE;
#pragma unroll
        for (int u = 0; u < XU; ++u) load16_to_lds(xsrc[u] + k0, dst + (wave * XU + u) * 8 * BK);
#pragma unroll
        for (int u = 0; u < WU; ++u) load16_to_lds(wsrc[u] + k0, dst + BM * BK + (wave * WU + u) * 8 * BK);
    };
    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    int foff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) foff[kk] = r * BK + (((4 * kk + c4) ^ ((r >> 1) & 7)) << 3);

    for (int i = 0; i < S - 1; ++i) gload(i, i);
    int stage = 0, fill = S - 1;
    for (int kt = 0; kt < nk; ++kt) {
        ring_barrier<(S - 2) * (XU + WU)>();   // k-tile kt has landed; everybody is done with the stage to be refilled
        gload(kt + S - 1, fill);
        const bf16* xs = lds + stage * STAGE + wm * WTM * BK;
        const bf16* ws = lds + stage * STAGE + BM * BK;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8 xf[TM], wf[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = !GLU ? wn * WTN + j * 16
                                : j < TN / 2 ? wn * (WTN / 2) + j * 16
                                             : BN / 2 + wn * (WTN / 2) + (j - TN / 2) * 16;
                wf[j] = *reinterpret_cast<const bf16x8*>(ws + row * BK + foff[kk]);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i) xf[i] = *reinterpret_cast<const bf16x8*>(xs + i * 16 * BK + foff[kk]);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf[i], acc[i][j], 0, 0, 0);
        }
        stage = stage + 1 == S ? 0 : stage + 1;
        fill = fill + 1 == S ? 0 : fill + 1;
    }
    ring_barrier<0>();   // the repeated loads must not land in the slabs
    GemmParams q = p;
    if (EPI == 2) q.C = reinterpret_cast<bf16*>(reinterpret_cast<float*>(p.C) + (size_t)blockIdx.y * p.M * p.N);
    store_tile<EPI, GROUPED, TM, TN>(q, acc, reinterpret_cast<float*>(smem) + wave * 32 * (WOUT + 4), lane, wm * WTM, tp.rows_valid,
                                     tp.m0, tp.n0 + wn * WOUT);
}

template <int BM, int BN, int WM, int WN, int S, int EPI, bool GROUPED>
static int launch_small(compact_ctx* ctx, GemmParams& p, hipStream_t s, int k_slices = 1) {
    constexpr int OUTN = EPI == 1 || EPI == 3 ? BN / 2 : BN;
    if (!GROUPED) p.n_mtiles = (int)((p.M + BM - 1) / BM);
    p.n_ntiles = (p.N + OUTN - 1) / OUTN;
    constexpr size_t smem = (size_t)S * (BM + BN) * GEMM_BK * sizeof(bf16);
    static_assert((size_t)WM * WN * 32 * (OUTN / WN + 4) * sizeof(float) <= smem, "the epilogue's slabs fit the ring");
    auto kern = gemm_bf16_small_kernel<BM, BN, WM, WN, S, EPI, GROUPED>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int64_t tiles = (int64_t)p.n_mtiles * p.n_ntiles;
    if (tiles == 0) return COMPACT_OK;
    kern<<<dim3((unsigned)tiles, (unsigned)k_slices), WM * WN * 64, smem, s>>>(p);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// How the 256 x 256 kernel cuts M rows: slots of 256 x 256 (a last row tile of more than 128 rows is one), and 128 x 256
// tiles of a bottom row tile of at most 128 rows.
struct LargeTiles {
    int64_t slots;
    int64_t bottom;
};
static LargeTiles large_tiles(int64_t M, int n_ntiles) {
    const int64_t rest = M % 256;
    return {(M / 256 + (rest > 128 ? 1 : 0)) * n_ntiles, rest > 0 && rest <= 128 ? n_ntiles : 0};
}

// n_full (plain products): slots of 256 x 256 that are whole tiles, see the kernel
template <int EPI, bool GROUPED>
static int launch_large(compact_ctx* ctx, GemmParams& p, int64_t n_full, int n_cus, hipStream_t s) {
    constexpr int OUTN = EPI == 1 ? 128 : 256;
    constexpr size_t smem = (size_t)9 * 128 * GEMM_BK * sizeof(bf16) + 2048;   // the larger ring; the epilogue's slabs fit in
    static_assert((size_t)8 * 32 * (OUTN / 4 + 4) * sizeof(float) <= smem, "the epilogue's slabs fit the ring");
    auto kern = gemm_bf16_kernel<EPI, GROUPED>;
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    p.n_ntiles = (p.N + OUTN - 1) / OUTN;
    int64_t wgs;
    if (GROUPED) {
        wgs = (int64_t)p.n_mtiles * p.n_ntiles;
    } else {
        const LargeTiles lt = large_tiles(p.M, p.n_ntiles);
        p.n_mtiles = (int)(lt.slots / p.n_ntiles);
        p.n_full = (int)std::min(n_full, lt.slots);
        wgs = p.n_full + 2 * (lt.slots - p.n_full) + lt.bottom;
        // Touches (tile_128) where the call is one round of half tiles: later rounds find the weights (N 4096 K 14336 at 4100
        // rows 442 -> 451 us).  From HBM, N 1088 .. 6144, K 2048 .. 14336 and 1024 .. 4600 rows, they gain 2 to 17 % (N 4096: K 2048
        // at 1400 rows 31.2 -> 27.2, K 14336 at 1100 rows 179 -> 148, at 1652 189 -> 163, at 2048 191 -> 176); weights
        // that the 256 MB cache still holds lose 1 to 8 % (K 2048 at 1100 rows 23.0 -> 24.3).  Whole prefills without them:
        // layer of 436 MB 0.996 .. 1.034 of the time with them, layers of 20 to 120 MB called again and again 0.980 .. 1.031.
        // K 1024 gains as much from HBM (18.7 -> 17.2) and loses as much from the cache (14.2 -> 14.8), and a layer so
        // narrow is more often there.
        p.touch = p.n_full == 0 && wgs <= n_cus && p.K >= 2048;
    }
    if (wgs == 0) return COMPACT_OK;
    kern<<<dim3((unsigned)wgs), 512, smem, s>>>(p);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Which tile.  Every form adds an output's products in the same order, so the choice changes no bit and may look at
// the number of rows.  The 256 x 256 kernel is priced at four cuts into whole and half tiles, by units that take the next
// tile when they are free (large_cost), the smaller forms by rounds of workgroups over the compute units x time of one tile
// (tile_cost); the time of a k-tile rises with the share u of busy units (power and L2 traffic).  Constants: microseconds per
// k-tile (idle chip + share of the load) and per tile, fitted to timings of the six forms apart; they know neither the shared
// launch of whole and half tiles nor the weight lines that half tiles touch ahead.  The pick against the best of the six
// forms and of half the slots as whole tiles, 360 calls (18 products, 64 .. 14336 columns, K 64 .. 14336, both
// epilogues, at 20 row counts from 65 to 20000, weights from HBM): of the 300 that take 8 us and more 0.6 % slower on average
// and five by 5 to 10.5 % (N 1088 K 2112 at 3700 rows 28.9 us as 128 x 64, 26.2 as half tiles; N 4096 K 14336 at 4600 rows
// 444, 414 with half the slots whole); the shorter ones, K of 64 to 512, 5 % on average and 1.1 us at most.
// Measured where the lines lie (us, 256 x 256 / 128 x 256): N 4096 K 14336 at 2048 rows 243 / 178, at 2500 rows 235 / 324
// (half tiles need a second round); N 6144 K 4096 at 2500 rows 91 / 109, at 3000 rows 154 / 136, and 126 mixed.
// Few rows, N 4096 K 14336: 65 rows 176 (256 x 256) / 176 / 113 (128 x 128) / 78 (64 x 128) / 76 (128 x 64) / 56
// (64 x 64); 400 rows 219 / 157 / 109 / 88 / 84 / 110; 1024 rows 246 / 151 / 131 / 187 / 185 / 219.
// ---------------------------------------------------------------------------
struct TileForm {
    int bm, bn;
    double t_idle, t_load, t_tile;
};
enum { TILE_256 = 0, TILE_128, TILE_128_128, TILE_128_64, TILE_64_128, TILE_64_64, TILE_FORMS };
static const TileForm tile_forms[TILE_FORMS] = {{256, 256, 1.00, 0.70, 4.8}, {128, 256, 0.75, 0.24, 2.7}, {128, 128, 0.55, 0.13, 1.7},
                                                {128, 64, 0.31, 0.03, 2.2},  {64, 128, 0.40, 0.04, 3.3},  {64, 64, 0.25, 0.05, 2.5}};

static double tile_cost(int form, double row_tiles, int N, int K, int epilogue, int n_cus) {
    const TileForm& f = tile_forms[form];
    const int outn = epilogue == 1 ? f.bn / 2 : f.bn;
    const double tiles = row_tiles * ((N + outn - 1) / outn);
    const double rounds = std::max(1.0, std::ceil(tiles / n_cus));
    return rounds * ((K / GEMM_BK) * (f.t_idle + f.t_load * tiles / (rounds * n_cus)) + f.t_tile);
}

// The 256 x 256 kernel: cost with n_full whole tiles, then `halves` 128 x 256 ones, each handed to the unit that is free
// first.  Workgroups are dealt to the eight XCDs round robin whatever their length, so the fullest XCD counts.
static double large_cost(int64_t n_full, int64_t halves, int K, int n_cus) {
    const TileForm &F = tile_forms[TILE_256], &H = tile_forms[TILE_128];
    const int nk = K / GEMM_BK, cus = std::max(1, n_cus / 8);
    const int64_t nf = (n_full + 7) / 8, nh = (halves + 7) / 8, busy = nf % cus, idle = cus - busy;
    double u = 1.0, end = 0;
    for (int pass = 0; pass < 2; ++pass) {   // the times depend on the average load, and it on the times
        const double tf = nk * (F.t_idle + F.t_load * u) + F.t_tile, th = nk * (H.t_idle + H.t_load * u) + H.t_tile;
        double ti = nf / cus * tf, tb = ti + tf;   // when the units with a tile less, and the others, are free
        end = busy ? tb : ti;
        for (int64_t left = nh; left > 0;) {
            double& t = ti <= tb ? ti : tb;
            left -= ti <= tb ? idle : busy;
            end = std::max(end, t += th);
        }
        u = std::min(1.0, (nf * tf + nh * th) / (end * cus));
    }
    return end;
}

static int pick_tile(int64_t M, int N, int K, int epilogue, int n_cus, int64_t* n_full) {
    // every slot a whole tile, whole rounds of them and the rest in halves, one round less, or halves only
    const int outn = epilogue == 1 ? 128 : 256, n_ntiles = (N + outn - 1) / outn;
    const LargeTiles lt = large_tiles(M, n_ntiles);
    const int64_t whole = lt.slots - lt.slots % n_cus;
    double best_cost = 0;
    for (const int64_t cut : {(int64_t)0, std::max<int64_t>(0, whole - n_cus), whole, lt.slots}) {
        const double c = large_cost(cut, 2 * (lt.slots - cut) + lt.bottom, K, n_cus);
        if (cut == 0 || c < best_cost) {
            best_cost = c;
            *n_full = cut;
        }
    }
    int best = *n_full > 0 ? TILE_256 : TILE_128;
    for (int form = TILE_128 + 1; form < TILE_FORMS; ++form) {
        const double c = tile_cost(form, (double)((M + tile_forms[form].bm - 1) / tile_forms[form].bm), N, K, epilogue, n_cus);
        if (c < best_cost) {
            best = form;
            best_cost = c;
        }
    }
    return best;
}

// Row-tile height of the grouped (per-expert) GEMMs of a routed layer over `rows` routed rows (256, 128 or 64): the cost
// as above for the gate/up and the down projection, with as many row tiles as evenly loaded experts would have.
int gemm_bf16_group_mtile(int64_t rows, int n_experts, int F, int d, int n_cus) {
    static const int forms[3] = {TILE_256, TILE_128, TILE_64_128};
    const double groups = (double)std::min<int64_t>(n_experts, std::max<int64_t>(rows, 1));
    const double per = rows / groups;
    int best = 256;
    double best_cost = 0;
    for (int i = 0; i < 3; ++i) {
        const int bm = tile_forms[forms[i]].bm;
        // a group of `per` rows on average: half a tile more than its rows fill, at least one
        const double row_tiles = groups * std::max(1.0, per / bm + 0.5);
        const double c = tile_cost(forms[i], row_tiles, F, d, 1, n_cus) + tile_cost(forms[i], row_tiles, d, F, 0, n_cus);
        if (i == 0 || c < best_cost) {
            best = bm;
            best_cost = c;
        }
    }
    return best;
}

template <int EPI, bool GROUPED>
static int launch_form(compact_ctx* ctx, int form, int64_t n_full, GemmParams& p, int n_cus, hipStream_t s) {
    switch (form) {
        case TILE_256: return launch_large<EPI, GROUPED>(ctx, p, n_full, n_cus, s);
        case TILE_128: return launch_large<EPI, GROUPED>(ctx, p, 0, n_cus, s);
        case TILE_64_128: return launch_small<64, 128, 2, 4, 6, EPI, GROUPED>(ctx, p, s);
        default: break;
    }
    if constexpr (!GROUPED) {
        switch (form) {
            case TILE_128_128: return launch_small<128, 128, 2, 4, 5, EPI, false>(ctx, p, s);
            case TILE_128_64: return launch_small<128, 64, 4, 2, 6, EPI, false>(ctx, p, s);
            case TILE_64_64: return launch_small<64, 64, 2, 2, 5, EPI, false>(ctx, p, s);
            default: break;
        }
    }
    return set_err(ctx, COMPACT_EINVAL, "unknown GEMM tile");
}

int launch_gemm_bf16(compact_ctx* ctx, const bf16* A, const bf16* B, const void* R, bool r_f32, bf16* C, int64_t M, int N,
                     int K, int epilogue, const GroupedArgs* grouped, hipStream_t s) {
    if (M == 0) return COMPACT_OK;
    if (K % GEMM_BK != 0 || N % 8 != 0) return set_err(ctx, COMPACT_ESHAPE, "bf16 GEMM needs K % 64 == 0 and N % 8 == 0");
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
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
        const int form = grouped->mtile == 256 ? TILE_256 : grouped->mtile == 128 ? TILE_128 : TILE_64_128;
        if (tile_forms[form].bm != grouped->mtile) return set_err(ctx, COMPACT_EINVAL, "no grouped GEMM of this row-tile height");
        return epilogue == 1 ? launch_form<1, true>(ctx, form, 0, p, n_cus, s) : launch_form<0, true>(ctx, form, 0, p, n_cus, s);
    }
    int64_t n_full = 0;
    const int form = pick_tile(M, N, K, epilogue, n_cus, &n_full);
    if (epilogue == 1) return launch_form<1, false>(ctx, form, n_full, p, n_cus, s);
    if (epilogue == 2) return launch_form<2, false>(ctx, form, n_full, p, n_cus, s);
    return launch_form<0, false>(ctx, form, n_full, p, n_cus, s);
}

// For the tests, not part of compact.h: the product in tile form `form` (TILE_FORMS: whole tiles and halves mixed, as many slots
// in either), or in the one the rule picks (-1); `picked` receives the rule's form.  And the row-tile height of the grouped
// products.
extern "C" int compact_test_gemm_form(compact_ctx* ctx, int32_t form, const void* a, const void* b, const void* r, void* c, int64_t M,
                                      int32_t N, int32_t K, int32_t epilogue, int32_t* picked, void* hip_stream) {
    if (!ctx || !a || !b || !c || !picked || M < 1 || N < 8 || N % 8 != 0 || K < GEMM_BK || K % GEMM_BK != 0 || form < -1 ||
        form > TILE_FORMS || (epilogue != 0 && epilogue != 1))
        return COMPACT_EINVAL;
    int n_cus = 0;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    GemmParams p{};
    p.X = (const bf16*)a;
    p.W = (const bf16*)b;
    p.R = (const bf16*)r;
    p.C = (bf16*)c;
    p.M = M;
    p.N = N;
    p.K = K;
    int64_t n_full = 0;
    *picked = pick_tile(M, N, K, epilogue, n_cus, &n_full);
    if (form < 0)
        form = *picked;
    else
        n_full = large_tiles(M, (N + (epilogue == 1 ? 127 : 255)) / (epilogue == 1 ? 128 : 256)).slots;
    if (form == TILE_FORMS) {
        form = TILE_256;
        n_full /= 2;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    return epilogue == 1 ? launch_form<1, false>(ctx, form, n_full, p, n_cus, s) : launch_form<0, false>(ctx, form, n_full, p, n_cus, s);
}
extern "C" int compact_test_group_mtile(compact_ctx* ctx, int64_t rows, int32_t n_experts, int32_t F, int32_t d, int32_t* mtile) {
    int n_cus = 0;
    if (!ctx || !mtile) return COMPACT_EINVAL;
    if (int rc = device_cu_count(ctx, &n_cus)) return rc;
    *mtile = gemm_bf16_group_mtile(rows, n_experts, F, d, n_cus);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Decode steps of 17 .. 64 rows: the 64 x 64 form as a weight stream.  Its ring keeps 64 KB of loads in flight per
// workgroup, two workgroups per CU, and the activations ride along by direct-to-LDS loads: the gate/up projection of the
// 8B-shaped layer streams its 235 MB in 50 us at 48 rows, what a plain read of them takes (kernels that stage the
// activations through registers: 59 us at 24 rows, 69 us at 64, against 49 and 55 us so).  Projections whose column tiles
// leave the chip idle are split over K into slices that depend on N and K alone: output and down projection together
// 33 us at 24 rows and 38 us at 64 (46 and 56 us before), the step at 64 rows 272 -> 243 us.
// ---------------------------------------------------------------------------
int gemm_rows64_slices(int N, int K) {
    const int tiles = (N + 63) / 64;
    return std::max(1, std::min(256 / tiles, (K + 511) / 512));
}

int launch_gemm_rows64(compact_ctx* ctx, const bf16* A, const bf16* B, float* partials, int M, int N, int K, hipStream_t s) {
    if (M < 1 || M > 64) return set_err(ctx, COMPACT_ESHAPE, "weight-streaming GEMM takes 1..64 activation rows");
    if (K % GEMM_BK != 0 || N % 8 != 0) return set_err(ctx, COMPACT_ESHAPE, "bf16 GEMM needs K % 64 == 0 and N % 8 == 0");
    GemmParams p{};
    p.X = A;
    p.W = B;
    p.C = reinterpret_cast<bf16*>(partials);
    p.M = M;
    p.N = N;
    p.K = K;
    return launch_small<64, 64, 2, 2, 5, 2, false>(ctx, p, s, gemm_rows64_slices(N, K));
}

int launch_swiglu_rows64(compact_ctx* ctx, const bf16* A, const bf16* B, const float* pre_scale, bf16* act, int M, int F, int K,
                         hipStream_t s) {
    if (M < 1 || M > 64) return set_err(ctx, COMPACT_ESHAPE, "weight-streaming GEMM takes 1..64 activation rows");
    if (K % GEMM_BK != 0 || F % 8 != 0) return set_err(ctx, COMPACT_ESHAPE, "bf16 GEMM needs K % 64 == 0 and N % 8 == 0");
    GemmParams p{};
    p.X = A;
    p.W = B;
    p.C = act;
    p.pre_scale = pre_scale;
    p.M = M;
    p.N = F;
    p.K = K;
    // Up to 32 rows: half the activation loads (rows past the last one are loaded again up to the 32nd, not the 64th); a stage is
    // 12 KB then, so one more fits beside a second workgroup.  N 2 * 14336, K 4096, 24 rows 48.5 -> 46.6 us.  Output and down
    // projection, a workgroup per CU, keep the 64-row tile: 31.9 us together against 31.5 with six stages of the lower one and
    // 33.4 with ten.
    if (M <= 32) return launch_small<32, 64, 1, 2, 6, 3, false>(ctx, p, s);
    return launch_small<64, 64, 2, 2, 5, 3, false>(ctx, p, s);
}
