// Varlen causal flash-style prefill attention (bf16 storage, MFMA).
// Every block attends only its own tokens; the packed batch is walked through
// a list of (block, 128-row query tile) items, block by block.
//
//  * a workgroup of 4 wavefronts = one query tile x one query head; a wavefront
//    owns 32 query rows and keeps Q^T in registers as the MFMA column operand.
//    Two (head_dim 64: three) workgroups per CU;
//  * K tiles [64 tok][hd] and V^T tiles [hd][64 tok] (the V slab is stored
//    transposed, so no transposition happens here) are staged by 16-byte
//    buffer loads that land in LDS directly (no register hop, no LDS stores),
//    in XOR-swizzled 16-byte chunks, two stages of either;
//  * S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_32x32x16_bf16.  Working
//    on the transposed problem puts one query row in one lane column, so the
//    online-softmax max/sum are in-lane reductions plus one cross-half
//    shuffle, and P^T feeds the second MFMA straight from the accumulator
//    registers: the MFMA rows of S^T are assigned to tokens such that each
//    lane's 8 accumulator values of a k-step are 8 consecutive tokens, which
//    is one 16-byte read of the V^T tile;
//  * the three parts of the work on 32 tokens (scores, softmax, output) run one
//    behind the other inside a wavefront: while the matrix pipe forms the scores
//    of half tile n + 1 and the output of n - 1, the vector ALU does the softmax of n,
//    MFMA by MFMA, in an order that is written out (the compiler's own leaves the
//    softmax behind the MFMAs).  Steps of 64 tokens instead of 32 keep 64 registers more
//    of scores and probabilities, which costs head_dim 64 its third wavefront per
//    SIMD (4 % of the time);
//  * the factor log2(e) / sqrt(hd) stands in the multiply-add before the exponential.
//    In the queries it would save head_dim 64 16 of 106 vector instructions per half tile
//    (2048 rows behind 16384, 64 + 8 heads, whole call of small products: 593 us instead of
//    644).  But where the rotation is slow a rotated query is close to a bf16 value, and the
//    factor takes it away from there before it is rounded: 0.5 to 3 % more error
//    against 64 bits, whatever the scores' size;
//  * causal tiles above the diagonal are skipped per wavefront; rows of the
//    V^T tile past the block's length are zeroed when staged.
// Bound: power.  16 blocks of 8192, 64 + 8 heads of 64: 9217 -> 8546 us (1.03
// PFLOP/s) with the matrix pipe 62 % busy (before: 54 %), clocks per tile and SIMD 942
// -> 830, but the clock falls with them; 8 blocks of 4096, 32 + 8 heads of 128: 1145
// -> 998 us (1.10 PFLOP/s), pipe 58 -> 69 %; 2048 rows behind 6144: 229 -> 221; blocks of
// 61 to 517 tokens: 26.2 -> 18.4 (inside the passes, one card).
// Before, head_dim 128 had workgroups of two heads whose wavefronts took turns at
// matrix and softmax phases between barriers, head_dim 64 ran scores, softmax and output
// one after the other in each of three wavefronts per SIMD.  The former, which staged K
// and V once for two heads, was faster in one kind of call: an even group of heads of 128 and one round of
// workgroups as long as each other (2048 rows behind 16384, 32 + 8 heads: whole
// call of small products 549 -> 564 to 576 us).
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "common.h"

#define KV_TILE 64
#define LOG2E 1.4426950408889634f

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Chunk swizzles.  The LDS has 64 banks of 4 bytes (256 bytes per cycle) and a
// 16-byte read is served 16 lanes at a time, so the 16 lanes must land in 16
// different 16-byte bank groups.  K-tile rows of 256 bytes (16 chunks) cover all
// groups by themselves: the 16 lanes read 16 different rows (a permutation of
// 0..15, +16), so the chunk index is XOR-ed with row % 16.  Rows of 128 bytes (8
// chunks: K at head_dim 64, every V^T tile) fill the banks two rows at a time:
// the chunk index is XOR-ed with (row / 2) % 8.
template <int CHUNKS>
__device__ __forceinline__ int swz(int row) { return CHUNKS == 16 ? (row & 15) : ((row >> 1) & 7); }

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ unsigned pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

// 16-byte buffer load whose result goes straight into LDS: lane l deposits its 16 bytes at
// lds_base + 16 * l (lds_base is wave-uniform) from byte base + voff of the buffer.  The range
// check (voff + 16 <= size) makes an out-of-range lane read zeros.  Offsets are
// 32-bit and the descriptor sits in scalar registers, so staging needs no 64-bit address arithmetic.
__device__ __forceinline__ void buf_load16_to_lds(__amdgpu_buffer_rsrc_t rsrc, void* lds_base, unsigned voff) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds_base, 16, voff, 0, 0, 0);
#else
    (void)rsrc, (void)lds_base, (void)voff;
#endif
}
// raw buffer descriptor over [p, p + bytes): stride 0, 32-bit data format
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// Waits until at most N of this wavefront's vector-memory operations are still in flight
// (they complete in order, so everything older has landed); LDS traffic is not waited for.
template <int N>
__device__ __forceinline__ void wait_vm() {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(N >= 0 && N < 64, "vector-memory counter is 6 bits");
    __builtin_amdgcn_sched_barrier(0);
    // simm16: vmcnt[3:0] | expcnt (7 = no wait) << 4 | lgkmcnt (15 = no wait) << 8 | vmcnt[5:4] << 14
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// Workgroup barrier that leaves global loads in flight: only this wavefront's LDS
// operations are waited for (its reads of a stage about to be refilled, its writes
// into a stage about to be read).
__device__ __forceinline__ void phase_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// Which (query tile, head) a workgroup takes.  Workgroups are dealt to the XCDs (an L2 each) round robin: XCD x takes KV heads
// x % xcd_heads + k xcd_heads, shared with the others of the same heads unit by unit (a unit: a query tile of a KV head, for
// all query heads of its group, side by side), and goes through one KV head's tiles before the next one's: what is in flight on
// an XCD reads the keys of a block or two (tiles of all blocks in flight everywhere: 8 blocks of 4096 7 % slower, 16 of 8192 at
// head_dim 64 5 %).  The sharers take their units forwards and backwards in turn, since a block's tiles
// come by length, and count them through all their heads: 40 + 5 heads of 128, a whole call of 512 rows behind 8192 183 us
// (263 in one direction and from the same XCD for every head, which left four of the eight idle), 4 blocks of 4096 863 (945).
struct PrefillPlace {
    int tile, kvh, g;   // kvh >= n_kv_heads: nothing to do
};
__host__ __device__ inline PrefillPlace prefill_place(int wg, int group, int n_qtiles, int xcd_heads) {
    const int x = wg % 8, share = 8 / xcd_heads, s = x / xcd_heads, round = wg / 8 / group;
    const int unit = round * share + (round & 1 ? share - 1 - s : s);
    return PrefillPlace{unit % n_qtiles, unit / n_qtiles * xcd_heads + x % xcd_heads, wg / 8 % group};
}
static int64_t prefill_workgroups(int n_q_heads, int n_kv_heads, int n_qtiles, int xcd_heads) {
    const int64_t share = 8 / xcd_heads, units = (int64_t)(n_kv_heads / xcd_heads) * n_qtiles;
    return 8 * (n_q_heads / n_kv_heads) * ((units + share - 1) / share);
}

// FAR: a block of the call has a slab of 4 GiB or more per KV head, whose V^T rows 32-bit offsets do not reach.
template <int HD, bool FAR>
__global__ __launch_bounds__(256, HD == 64 && !FAR ? 3 : 2) void attn_prefill_bf16_kernel(const BlockMeta* __restrict__ meta,
                                                                     const TileItem* __restrict__ qtiles,
                                                                     const bf16* __restrict__ qkv,
                                                                     const bf16* __restrict__ kbase,
                                                                     const bf16* __restrict__ vbase, bf16* __restrict__ o,
                                                                     int Hq, int Hkv, int n_qtiles, int xcd_heads, float scale_log2) {
    constexpr int KK = HD / 16;        // k16 steps of S^T
    constexpr int DT = HD / 32;        // 32-row tiles of O^T
    constexpr int KCH = HD / 8;        // 16-byte chunks per K row
    constexpr int KTILE = KV_TILE * HD;   // elements of a K tile == elements of a V^T tile
    constexpr int NW = 4;                 // wavefronts that stage a tile
    constexpr int NLD = KTILE / 8 / (NW * 64);  // chunks per thread per tile
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* lds = reinterpret_cast<bf16*>(smem);  // [2 K tiles | 2 V^T tiles]

    const PrefillPlace pl = prefill_place(blockIdx.y * gridDim.x + blockIdx.x, Hq / Hkv, n_qtiles, xcd_heads);
    if (pl.kvh >= Hkv) return;
    const int kvh = pl.kvh, head = kvh * (Hq / Hkv) + pl.g;
    const TileItem it = qtiles[pl.tile];
    const BlockMeta bm = meta[it.block];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int ld = (Hq + 2 * Hkv) * HD;
    const int len = bm.prior + bm.len;   // cache rows once this call's rows are in
    const int prior = bm.prior;          // query row i of the call is cache row prior + i

    const bf16* kslab = kbase + bm.slab + (size_t)kvh * bm.capacity * HD;
    const bf16* vslab = vbase + bm.slab + (size_t)kvh * HD * bm.capacity;

    // ---- Q^T operand: lane (q = r, h) holds Q[q][kk*16 + h*8 .. +7] -----------
    const int qrow = prior + it.row0 + wave * 32 + r;   // as a cache row
    const bf16* qp = qkv + (size_t)(bm.row0 + min(qrow, len - 1) - prior) * ld + head * HD + h * 8;
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qp + kk * 16);

    floatx16 oacc[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[d][e] = 0.f;
    float l_run = 0.f, l_even = 0.f;   // sums of the probabilities: of whole tiles, and of a tile's first half
    float neg_m = 0.f;   // the scaling reference, negated

    const int q_hi_wg = min(prior + it.row0 + PREFILL_QTILE, len) - 1;   // last query row of the workgroup
    const int q_lo_wave = prior + it.row0 + wave * 32;                     // first query row of this wave
    const int n_tiles = q_hi_wg / KV_TILE + 1;
    const int n_mine = min(n_tiles, (q_lo_wave + 31) / KV_TILE + 1);     // tiles not wholly above this wave's diagonal

    // ---- staging: 16-byte buffer loads that land in LDS directly ---------------------
    // A wave-instruction fills 64 consecutive 16-byte chunks of a tile; chunk L of the K tile is
    // (row L / KCH, position L % KCH) and holds the row's chunk (L % KCH) ^ swz(row), chunk L of the
    // V^T tile likewise with 8 chunks per row: each lane picks the global address that belongs in
    // its slot.  Wavefront w issues instructions w, w + NW, ...; nothing passes through registers.
    unsigned koff[NLD], voff[NLD];   // byte offsets inside a tile's source rows, fixed per lane
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int L = (i * NW + wave) * 64 + lane;
        const int krow = L / KCH, kc = (L % KCH) ^ swz<KCH>(krow);
        koff[i] = (unsigned)(krow * HD + kc * 8) * 2u;
        const int vrow = L >> 3, vc = (L & 7) ^ swz<8>(vrow);
        voff[i] = (unsigned)(vrow * bm.capacity + vc * 8) * 2u;
    }
    const unsigned slab_bytes = (unsigned)bm.capacity * HD * 2u;   // one KV head's K slab, and its V^T slab (below 4 GiB)
    // A tile has descriptors of its own, from its first byte to the slab's end: K rows and V^T columns past the slab read
    // zeros, and so does a tile past the last one; rows past the block's end inside the slab read whatever is there (their
    // scores are masked, their V^T columns are zeroed by fix_tail).
    // FAR: K tiles have descriptors of their own 64 rows (fewer at the slab's end), V^T chunks go by 64-bit addresses, those
    // past a row's end by that of the row's last chunk (zeroed by fix_tail like the others).
    auto issue_k = [&](int kt, int i) __attribute__((always_inline)) {
        if constexpr (FAR) {
            const unsigned bytes = kt < n_tiles ? (unsigned)min(KV_TILE, bm.capacity - kt * KV_TILE) * HD * 2u : 0u;
            buf_load16_to_lds(raw_buffer(kslab + (size_t)kt * KTILE, bytes), lds + (kt & 1) * KTILE + (i * NW + wave) * 64 * 8, koff[i]);
            return;
        }
        const int off = kt * KV_TILE * HD;
        const __amdgpu_buffer_rsrc_t rs = raw_buffer(kslab + off, kt < n_tiles ? slab_bytes - 2u * off : 0u);
        buf_load16_to_lds(rs, lds + (kt & 1) * KTILE + (i * NW + wave) * 64 * 8, koff[i]);
    };
    auto issue_v = [&](int kt, int i) __attribute__((always_inline)) {   // kt < n_tiles
        if constexpr (FAR) {
            const int vrow = ((i * NW + wave) * 64 + lane) >> 3, col = kt * KV_TILE + (((lane & 7) ^ swz<8>(vrow)) << 3);
            load16_to_lds(vslab + (size_t)vrow * bm.capacity + min(col, bm.capacity - 8),
                          lds + (2 + (kt & 1)) * KTILE + (i * NW + wave) * 64 * 8);
            return;
        }
        const int off = kt * KV_TILE;
        const __amdgpu_buffer_rsrc_t rs = raw_buffer(vslab + off, kt < n_tiles ? slab_bytes - 2u * off : 0u);
        buf_load16_to_lds(rs, lds + (2 + (kt & 1)) * KTILE + (i * NW + wave) * 64 * 8, voff[i]);
    };
    // After a wavefront's own loads of a LAST tile have landed: zero the V^T entries of tokens past
    // the block's end (whatever the slab holds there must not reach the MFMA; their probabilities are 0).
    auto fix_tail = [&](int kt) {
        const int kv0 = kt * KV_TILE;
        if (__builtin_expect(kv0 + KV_TILE <= len || kt >= n_tiles, 1)) return;
        bf16* vs = lds + (2 + (kt & 1)) * KTILE;
        const int ln = here(lane);
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int L = (i * NW + wave) * 64 + ln;
            const int vrow = L >> 3, vc = (L & 7) ^ swz<8>(vrow);
            if (kv0 + vc * 8 + 8 > len) {
                bf16x8 v = *reinterpret_cast<bf16x8*>(vs + (size_t)L * 8);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (kv0 + vc * 8 + j >= len) v[j] = (bf16)0.f;
                *reinterpret_cast<bf16x8*>(vs + (size_t)L * 8) = v;
            }
        }
    };

    // token of MFMA row i of S^T tile tt: tt*32 + pi(i); pi keeps each lane's
    // accumulator values of one k-step on 8 consecutive tokens
    const int pi_r = (r >> 4) * 16 + ((r >> 2) & 1) * 8 + ((r >> 3) & 1) * 4 + (r & 3);

    // Scores go in halves of 32 tokens: S^T of half n holds query column r, token 32 n + (e/8)*16 + h*8 + (e%8).  Two halves
    // are alive, even ones in se, odd ones in so; likewise their P^T, the column operand of the second MFMA (eight bf16).
    floatx16 se, so;
    uintx4 pe[2], po[2];

    // LDS byte offsets of the fragments of a tile: K row pi_r (the second half 32 rows on, same swizzle), V^T row r
    int kfo[KK], vfo[4];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kfo[kk] = 2 * (pi_r * HD + (((kk * 2 + h) ^ swz<KCH>(pi_r)) << 3));
#pragma unroll
    for (int u = 0; u < 4; ++u) vfo[u] = 2 * (r * KV_TILE + (((u * 2 + h) ^ swz<8>(r)) << 3));
    auto k_frag = [&](int stage, int tt, int kk) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(smem + kfo[kk] + 2 * (stage * KTILE + tt * 32 * HD));
    };
    auto v_frag = [&](int stage, int d, int u) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x8*>(smem + vfo[u] + 2 * ((2 + stage) * KTILE + d * 32 * KV_TILE));
    };
    auto zeros = []() __attribute__((always_inline)) {
        floatx16 z;
#pragma unroll
        for (int e = 0; e < 16; ++e) z[e] = 0.f;
        return z;
    };
    // probabilities of a half against the reference as it stands; `ps` and the lane's 16 values
    auto prob = [&](float x) __attribute__((always_inline)) {
        return __builtin_amdgcn_exp2f(__builtin_fmaf(x, scale_log2, neg_m));
    };
    auto probs = [&](float ps, const floatx16& s, uintx4 (&p)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const float a = prob(s[e]), b = prob(s[e + 1]);
            ps += a;
            ps += b;
            p[e >> 3][(e >> 1) & 3] = pack_bf16x2(a, b);
        }
        return ps;
    };
    auto mask = [&](int n, floatx16& s) __attribute__((always_inline)) {
        if (__builtin_expect(n * 32 + 31 <= q_lo_wave, 1)) return;   // wholly below the wavefront's diagonal
        const int q = here(qrow) - n * 32 - h * 8;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if ((e >> 3) * 16 + (e & 7) > q) s[e] = -INFINITY;
    };
    // The running maximum is only a scaling reference.  The common case takes the probabilities against the reference as
    // it stands and looks at nothing but their sum: while every lane's sum of a tile's 32 values stays below 2^12, fp32 sums and
    // bf16 probabilities carry them without loss and the half's maximum is never formed.  Otherwise
    // the exact maximum is taken, the reference moves there, the accumulators are rescaled and the probabilities are
    // formed again.  A first half takes the maximum of its whole tile (its second half's scores, n + 1, are in `other`), so that
    // the tile's largest weight is 1, which is not rounded: with the half's own, 0.1 to 1 % more error against 64 bits, most
    // by the first tile.
    // A tile's values are summed one after the other through both halves (`ps`: an odd half's sum has begun with l_even) before
    // they join those of the tiles before.
    // (Query columns past the block's end see unmasked cache rows past it -- whatever the slab holds -- and must not take
    // part in the decision: a row's bits may depend on its own block only.)
    auto settle = [&](int n, float ps, bool odd, bool first, const floatx16& s, floatx16& other, uintx4 (&p)[2])
                      __attribute__((always_inline)) {
        if (__builtin_expect(first || __any(!(ps < 4096.0f) && qrow < len), 0)) {
            float mx = -INFINITY;
            if (!odd) mask(n + 1, other);
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, odd ? s[e] : fmaxf(s[e], other[e]));
            mx = __builtin_fmaf(fmaxf(mx, __shfl_xor(mx, 32, 64)), scale_log2, neg_m);
            const float up = first ? mx : fmaxf(mx, 0.f);   // finite: half 0 holds token 0 <= every query row
            const float corr = first ? 1.f : __builtin_amdgcn_exp2f(-up);
            l_run *= corr;
            neg_m -= up;
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int e = 0; e < 16; ++e) oacc[d][e] *= corr;
            ps = probs(odd ? l_even * corr : 0.f, s, p);
        }
        if (odd)
            l_run += ps;
        else
            l_even = ps;
    };

    // Step J of a wavefront, with K of tile J and V^T of tile J - 1, is twice (first for n = 2J - 1, then for n = 2J) QK^T of
    // half n + 1, softmax of half n and PV of half n - 1, which do not depend on each other.  The instructions stand in the
    // order in which they are to issue: MFMAs of the two products in turn, per MFMA an operand read AHEAD fragments before its
    // use and a share of the softmax (PRE MFMAs ahead: the first operands are on their way meanwhile), and at the step's
    // start the staging loads of the next one.
    constexpr int NM = 2 * KK, AHEAD = 4, PER = 16 / NM, PRE = 2 / PER;
    static_assert(KK == 2 * DT, "as many MFMAs in either product");
    bf16x8 fr[2 * NM];
    auto half_step = [&](auto ptag, auto stag, int J, floatx16& sc, floatx16& sn, const uintx4 (&pp)[2], uintx4 (&pn)[2])
                         __attribute__((always_inline)) {
        constexpr int part = decltype(ptag)::value, stage = decltype(stag)::value;   // stage of K; V^T lies in the other one
        auto read = [&](int g) __attribute__((always_inline)) {
            const int i = g % NM, tt = g / NM, m = i / 2;
            fr[g] = i & 1 ? v_frag(1 - stage, m % DT, 2 * tt + m / DT) : k_frag(stage, tt, m);
        };
        float ps = part == 0 ? l_even : 0.f, pv[16];   // part 0 is an odd half
        auto add = [&](int e) __attribute__((always_inline)) {
            ps += pv[e];
            if (e & 1) pn[e >> 3][(e >> 1) & 3] = here((int)pack_bf16x2(pv[e - 1], pv[e]));   // not sunk below the branch
        };
        if (part == 0) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) read(i);
        }
        mask(2 * J - 1 + part, sc);
#pragma unroll
        for (int e = 0; e < PRE * PER; ++e) pv[e] = prob(sc[e]);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int g = part * NM + i, m = i / 2;
            __builtin_amdgcn_sched_barrier(0);
            if (g + AHEAD < 2 * NM) read(g + AHEAD);
            if (i & 1)
                oacc[m % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], __builtin_bit_cast(bf16x8, pp[m / DT]), oacc[m % DT], 0, 0, 0);
            else
                sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], qf[m], m ? sn : zeros(), 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = (i + PRE) * PER; e < (i + PRE + 1) * PER && e < 16; ++e) pv[e] = prob(sc[e]);
#pragma unroll
            for (int e = i ? (i + PRE - 1) * PER : 0; e < (i + PRE) * PER && e < 16; ++e) add(e);
            if (part == 0 && i < 2 * NLD) {
                if (i < NLD)
                    issue_k(J + 1, i);
                else
                    issue_v(J, i - NLD);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        settle(2 * J - 1 + part, ps, part == 0, false, sc, sn, pn);
    };
    auto issue = [&](int J) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            issue_k(J + 1, i);
            issue_v(J, i);
        }
    };
    auto landed = [&](int J) __attribute__((always_inline)) {   // end of step J: what it requested is there
        wait_vm<0>();
        fix_tail(J);
        phase_barrier();
    };
    auto step = [&](auto stag, int J) __attribute__((always_inline)) {
        half_step(std::integral_constant<int, 0>{}, stag, J, so, se, pe, po);
        half_step(std::integral_constant<int, 1>{}, stag, J, se, so, po, pe);
        landed(J);
    };
#pragma unroll
    for (int i = 0; i < NLD; ++i) issue_k(0, i);
    issue(0);
    wait_vm<2 * NLD>();
    phase_barrier();
#pragma unroll
    for (int m = 0; m < KK; ++m) {
        se = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(0, 0, m), qf[m], m ? se : zeros(), 0, 0, 0);
        so = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(0, 1, m), qf[m], m ? so : zeros(), 0, 0, 0);
    }
    mask(0, se);
    settle(0, 0.f, false, true, se, so, pe);
    landed(0);
    int J = 1;
#pragma unroll 1
    for (; J + 1 < n_mine; J += 2) {
        step(std::integral_constant<int, 1>{}, J);
        step(std::integral_constant<int, 0>{}, J + 1);
    }
    if (J < n_mine) step(std::integral_constant<int, 1>{}, J++);
    // the last step: no scores to form, and its second half may lie above the diagonal
    if (J < n_tiles) issue(J);
    {
        const int stage = (J - 1) & 1, n = 2 * J - 1;
        const bool more = n * 32 <= q_lo_wave + 31;
        float ps = l_even;
        if (more) {
            mask(n, so);
            ps = probs(ps, so, po);
        }
#pragma unroll
        for (int m = 0; m < KK; ++m)
            oacc[m % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(stage, m % DT, m / DT), __builtin_bit_cast(bf16x8, pe[m / DT]),
                                                                   oacc[m % DT], 0, 0, 0);
        if (more) {
            settle(n, ps, true, false, so, se, po);
#pragma unroll
            for (int m = 0; m < KK; ++m)
                oacc[m % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(stage, m % DT, 2 + m / DT), __builtin_bit_cast(bf16x8, po[m / DT]),
                                                                       oacc[m % DT], 0, 0, 0);
        } else {
            l_run += ps;
        }
    }
    if (J < n_tiles) landed(J++);
#pragma unroll 1
    for (; J < n_tiles; ++J) {   // the other wavefronts' last tiles
        issue(J);
        landed(J);
    }

    // ---- normalise and store: lane (q = r) holds elements d*32 + (e/4)*8 + h*4 + (e%4) ----
    l_run += __shfl_xor(l_run, 32, 64);
    if (qrow < len) {
        const float inv = 1.0f / l_run;
        bf16* op = o + (size_t)(bm.row0 + qrow - prior) * Hq * HD + head * HD;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (bf16)(oacc[d][g * 4 + e] * inv);
                *reinterpret_cast<bf16x4*>(op + d * 32 + g * 8 + h * 4) = v;
            }
    }
}

template <int HD, bool FAR>
static int launch_prefill_variant(compact_ctx* ctx, const BlockMeta* d_meta, const TileItem* d_qtiles, int n_qtiles,
                                  const bf16* qkv, const bf16* d_k, const bf16* d_v, bf16* o, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    auto kern = attn_prefill_bf16_kernel<HD, FAR>;
    const size_t smem = (size_t)4 * KV_TILE * HD * sizeof(bf16);
    static bool attr_set = false;
    if (!attr_set) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int xcd_heads = std::gcd(8, c.n_kv_heads);
    // One grid dimension takes 2^32 threads and drops what is over without an error: beyond 2^20 workgroups the grid has rows of as
    // many, a multiple of 8, so that a workgroup's number still says which XCD it is dealt to.
    const int64_t wgs = prefill_workgroups(c.n_q_heads, c.n_kv_heads, n_qtiles, xcd_heads), row = 1 << 20;
    if (wgs > INT32_MAX - row) return set_err(ctx, COMPACT_ESHAPE, "too many query tiles and heads for one call");
    const dim3 grid((unsigned)std::min(wgs, row), (unsigned)((wgs + row - 1) / row));
    kern<<<grid, 256, smem, s>>>(d_meta, d_qtiles, qkv, d_k, d_v, o, c.n_q_heads, c.n_kv_heads, n_qtiles, xcd_heads,
                                 LOG2E / sqrtf((float)c.head_dim));
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// `far`: see the kernel.  Slabs below 4 GiB keep the descriptors, which need no 64-bit address per lane.
int launch_attn_prefill_bf16(compact_ctx* ctx, const BlockMeta* d_meta, int max_capacity, const TileItem* d_qtiles, int n_qtiles,
                             const bf16* qkv, const bf16* d_k, const bf16* d_v, bf16* o, hipStream_t s) {
    if (n_qtiles == 0) return COMPACT_OK;
    const int hd = ctx->cfg.head_dim;
    const bool far = (int64_t)max_capacity * hd * (int64_t)sizeof(bf16) >= (int64_t)1 << 32;
    auto launch = hd == 128 ? (far ? launch_prefill_variant<128, true> : launch_prefill_variant<128, false>)
                            : (far ? launch_prefill_variant<64, true> : launch_prefill_variant<64, false>);
    return launch(ctx, d_meta, d_qtiles, n_qtiles, qkv, d_k, d_v, o, s);
}

// For the tests, not part of compact.h: query tile, KV head and query head of the workgroups 0 .. n - 1 of a call with n_qtiles
// query tiles (KV heads past the last one: nothing to do); returns the number of the call's workgroups.
extern "C" int64_t compact_test_prefill_place(int32_t n_q_heads, int32_t n_kv_heads, int32_t n_qtiles, int32_t n, int32_t* out) {
    const int xcd_heads = std::gcd(8, n_kv_heads), group = n_q_heads / n_kv_heads;
    for (int i = 0; i < n; ++i) {
        const PrefillPlace pl = prefill_place(i, group, n_qtiles, xcd_heads);
        out[3 * i] = pl.tile;
        out[3 * i + 1] = pl.kvh;
        out[3 * i + 2] = pl.kvh * group + pl.g;
    }
    return prefill_workgroups(n_q_heads, n_kv_heads, n_qtiles, xcd_heads);
}
