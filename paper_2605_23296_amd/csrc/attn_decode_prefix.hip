// Decode attention of the prefix-aware layout (paper Sec. IV, Dispatch: worker
// k's prompt is blocks 1..k, so every worker's cache prefix is a prefix of the
// one shared cache of the whole history): worker b attends rows
// 0 .. prefix_len[b]-1 of the SHARED slab plus its own private tail.
//
// Cascade over the shared rows: a work item is a chunk of 128 .. 1536 rows of
// the shared slab (by the length of the history: short ones need the workgroups, long
// ones the fewer records) together with the workers whose prefix reaches into it (a
// suffix of the workers, prefixes being nested; at most PFX_COLS query columns =
// workers x heads of the KV group, more workers make further items over the same
// rows).  A worker's private tail is cut into one-worker items of the same kernel.
// Every item leaves one record (un-normalised output, max, sum) per (worker, head); a
// second kernel merges a worker's records.
//
//  * a workgroup of 8 wavefronts walks its item in tiles of 32 rows, two workgroups
//    per CU.  K and V^T land in LDS by direct 16-byte loads (swizzled slots), read
//    once from memory for all columns: V^T two tiles at a time (whole 128-byte lines
//    of the transposed slab) in a ring of three pairs, K tile by tile in a ring of
//    four (at head_dim 64 pairs as well);
//  * every wavefront owns 16 query columns and keeps its online softmax and output
//    rows in registers: S^T = K Q^T with the K rows assigned to MFMA rows such that
//    a lane ends up with 8 consecutive rows of one column, which is the P^T operand
//    of O^T += V^T P^T without a trip through LDS.  Nothing is exchanged between
//    wavefronts, one barrier per tile;
//  * the walk must not spill: a scratch reload waits for every load in flight and
//    drains the ring (236 us instead of 96), hence here() in the rare branches;
//  * bound: HBM (a step reads every shared row once).  24 workers over 98304 rows
//    (403 MB): 119 -> 96 us, the merge of its records 25.6 -> 12.8 us,
//    with items of 1536 rows 7.5; 8 workers over
//    32768 rows: both together 52.7 -> 49.8 us.  (Before: 256-row items, the rows
//    split over the wavefronts, maxima and probabilities exchanged through LDS, three
//    barriers per 16 columns; twice the records.)  Loads alone take 87 us.
#include "common.h"

#define LOG2E 1.4426950408889634f
#define PFX_WAVES 8
#define PFX_TILE 32
#define PFX_PAIR (2 * PFX_TILE)
#define PFX_VSLOTS 3
static_assert(PFX_COLS == PFX_WAVES * 16, "one 16-column MFMA group per wavefront");

__device__ __forceinline__ float pfx_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max / sum over the four lanes that share lane % 16, without a trip through LDS
template <bool MAX>
__device__ __forceinline__ float over_rows(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
    // permlane32_swap(x, y) exchanges the upper half of x with the lower half of y, permlane16_swap likewise rows of 16
    // lanes; y is a copy that the compiler must not know to be one (it takes both results for the same value otherwise)
    unsigned p = __builtin_bit_cast(unsigned, x), q = p;
    asm("" : "+v"(q));
    auto a = __builtin_amdgcn_permlane32_swap(p, q, false, false);
    const float lo = __builtin_bit_cast(float, (unsigned)a[0]), hi = __builtin_bit_cast(float, (unsigned)a[1]);
    x = MAX ? fmaxf(lo, hi) : lo + hi;
    p = q = __builtin_bit_cast(unsigned, x);
    asm("" : "+v"(q));
    auto b = __builtin_amdgcn_permlane16_swap(p, q, false, false);
    const float e = __builtin_bit_cast(float, (unsigned)b[0]), o = __builtin_bit_cast(float, (unsigned)b[1]);
    x = MAX ? fmaxf(e, o) : e + o;
#endif
    return x;
}

// Waits until at most N of this wavefront's loads are in flight and its LDS reads have returned, then joins the barrier.
template <int N>
__device__ __forceinline__ void pfx_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(N >= 0 && N < 16, "count fits the low four bits");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(N | (7 << 4) | (0 << 8));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}

template <int HD>
__global__ __launch_bounds__(PFX_WAVES * 64, 4) void attn_decode_prefix_kernel(
    const BlockMeta* __restrict__ tail_meta, const BlockMeta shared, const PrefixItem* __restrict__ items, int step,
    const bf16* __restrict__ q, const bf16* __restrict__ kshared, const bf16* __restrict__ vshared, const bf16* __restrict__ ktail,
    const bf16* __restrict__ vtail, float* __restrict__ records, int64_t total_recs, int Hq, int Hkv, float scale_log2) {
    constexpr int KS = HD / 32;               // k-steps of the QK product
    constexpr int DT = HD / 16;               // 16-row tiles of O^T
    constexpr int KCH = HD / 8;               // 16-byte chunks per K row
    constexpr int KT = HD == 128 ? PFX_TILE : PFX_PAIR;   // rows of a K load: 8 KB, one instruction per wavefront, either way
    constexpr int KSLOTS = HD == 128 ? 4 : 3;
    constexpr int VE = PFX_PAIR * HD, KE = KT * HD;       // elements of a V^T pair, of a K slot
    constexpr int NV = VE / 512 / PFX_WAVES;              // 1 KB load instructions per wavefront for a V^T pair
    static_assert(KE / 512 == PFX_WAVES, "one K load instruction per wavefront");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* vlds = reinterpret_cast<bf16*>(smem);           // [slot][HD][64 tokens]
    bf16* klds = vlds + PFX_VSLOTS * VE;                  // [slot][KT rows][HD]

    const PrefixItem it = items[blockIdx.x];
    const int kvh = blockIdx.y;
    const int G = Hq / Hkv;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, c = lane >> 4;

    const bf16 *kslab, *vslab;
    int cap, n_rows;   // rows of the item that exist at all
    if (it.tail) {
        const BlockMeta bm = tail_meta[it.w0];
        n_rows = min(bm.len + step + 1 - it.row0, PREFIX_TAIL_CHUNK);
        if (n_rows <= 0) return;   // a tail chunk this step does not reach yet
        cap = bm.capacity;
        kslab = ktail + bm.slab + (size_t)kvh * cap * HD;
        vslab = vtail + bm.slab + (size_t)kvh * HD * cap;
    } else {
        n_rows = it.n_rows;
        cap = shared.capacity;
        kslab = kshared + shared.slab + (size_t)kvh * cap * HD;
        vslab = vshared + shared.slab + (size_t)kvh * HD * cap;
    }
    const int n_tiles = (n_rows + PFX_TILE - 1) / PFX_TILE;
    const int last_row = it.row0 + n_rows - 1;

    // ---- this wavefront's 16 query columns: operand lane (r, c) holds q[column r][s*32 + c*8 .. +7] ----
    const int ncols = it.nw * G;
    const int col = wave * 16 + r;
    const bool active = wave * 16 < ncols;
    const int col_c = min(col, ncols - 1);
    const int wk = it.w0 + col_c / G;
    bf16x8 qf[KS];
    {
        const bf16* qp = q + ((size_t)wk * Hq + kvh * G + col_c % G) * HD + c * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + s * 32);
    }
    // rows of the item the column may see, and the least of the wavefront's columns (tiles below it need no mask)
    const int lim = col < ncols ? (it.tail ? n_rows : min(n_rows, tail_meta[wk].pos_offset - it.row0)) : 0;
    int least = lim;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) least = min(least, __shfl_xor(least, o, 64));
    least = __builtin_amdgcn_readfirstlane(least);

    // ---- staging: instruction n of a load fills LDS chunks 64 n .. 64 n + 63 of its slot (K rows of KCH chunks, V^T rows
    // of 8).  The 16 lanes of an operand read touch rows {0-3, 8-11, 16-19, 24-27} (+ 4, + 32) of K, 16 consecutive rows
    // of V^T; the chunk swizzles spread those over the 64 banks.
    auto swz_k = [](int row) { return KCH == 16 ? (row & 3) | ((row >> 3) & 3) << 2 : ((row >> 1) & 1) | ((row >> 3) & 3) << 1; };
    auto swz_v = [](int d) { return (d >> 1) & 7; };
    const int krow = (wave * 64 + lane) / KCH, kch = ((lane % KCH) ^ swz_k(krow)) * 8;
    const int vd0 = (wave * NV * 64 + lane) >> 3, vc = lane & 7;   // V^T rows vd0, vd0 + 8
    auto issue_k = [&](int kt, int slot) {   // rows past the item: its last row
        load16_to_lds(kslab + (size_t)min(it.row0 + kt * KT + krow, last_row) * HD + kch, klds + slot * KE + wave * 512);
    };
    auto issue_v = [&](int pair, int slot) {   // columns past the slab: its last ones
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int d = vd0 + 8 * i;
            load16_to_lds(vslab + (size_t)d * cap + min(it.row0 + pair * PFX_PAIR + ((vc ^ swz_v(d)) << 3), cap - 8),
                          vlds + slot * VE + (wave * NV + i) * 512);
        }
    };

    float m_run = -INFINITY, l_run = 0.f;   // of column r; l_run: this lane's share
    floatx4 oacc[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) oacc[i] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Loads in flight at the wait of a tile (what is younger than its own): head_dim 128, order V0 K0 K1 V1 K2 | V2 K3 | K4 |
    // V3 K5 | ...: a V^T pair (NV) and two K tiles; head_dim 64, order V0 K0 V1 K1 | V2 K2 | - | V3 K3 ...: one pair of each
    // before an even tile, two before an odd one (whose rows came with the even one).
    issue_v(0, 0);
    issue_k(0, 0);
    if (HD == 128) issue_k(1, 1);
    issue_v(1, 1);
    issue_k(HD == 128 ? 2 : 1, HD == 128 ? 2 : 1);
    int vslot = 0, kslot = 0;
    for (int tile = 0; tile < n_tiles; ++tile) {
        const int odd = tile & 1;
        // the tile has landed; everybody is done with the slots to be refilled
        if (HD == 128)
            pfx_barrier<NV + 2>();
        else if (odd)
            pfx_barrier<2 * (NV + 1)>();
        else
            pfx_barrier<NV + 1>();
        if (!odd) issue_v((tile >> 1) + 2, vslot == 0 ? 2 : vslot - 1);
        if (HD == 128)
            issue_k(tile + 3, (kslot + 3) & 3);
        else if (!odd)
            issue_k((tile >> 1) + 2, kslot == 0 ? 2 : kslot - 1);
        const bf16* ks = klds + kslot * KE + (HD == 128 ? 0 : odd * PFX_TILE * HD);
        bf16* vs = vlds + vslot * VE;
        const int rows_left = n_rows - tile * PFX_TILE;
        if (rows_left < PFX_TILE) {   // the last tile: V^T columns past the item's end must not reach the MFMA, whatever their bits
            for (int L = here(t); L < HD * 4; L += PFX_WAVES * 64) {
                const int d = L >> 2, ch = L & 3;
                bf16* vp = vs + d * PFX_PAIR + (((odd * 4 + ch) ^ swz_v(d)) << 3);
                bf16x8 v = *reinterpret_cast<bf16x8*>(vp);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (8 * ch + j >= rows_left) v[j] = (bf16)0.f;
                *reinterpret_cast<bf16x8*>(vp) = v;
            }
            pfx_barrier<15>();
        }
        if (active) {
            // all operand reads of a product go out before its first MFMA (the compiler would wait for every pair)
            floatx4 sacc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
            bf16x8 kf[KS][2];
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) {
                    const int row = 8 * (r >> 2) + 4 * tt + (r & 3);
                    kf[s][tt] = *reinterpret_cast<const bf16x8*>(ks + row * HD + (((s * 4 + c) ^ swz_k(row)) << 3));
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) sacc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][tt], qf[s], sacc[tt], 0, 0, 0);
            // sacc[tt][e]: column r, tile row 8c + 4tt + e
            float sv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) sv[j] = sacc[j >> 2][j & 3] * scale_log2;
            if (tile * PFX_TILE + PFX_TILE > least) {
                const int left = lim - tile * PFX_TILE - 8 * here(c);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (j >= left) sv[j] = -INFINITY;
            }
            float mx = sv[0];
#pragma unroll
            for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sv[j]);
            mx = over_rows<true>(mx);
            {
                const float m_new = fmaxf(m_run, mx);
                const float alpha = pfx_exp2(m_run - (m_new == -INFINITY ? 0.f : m_new));
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int i = 0; i < DT; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) oacc[i][e] *= alpha;
            }
            const float m_use = m_run == -INFINITY ? 0.f : m_run;   // a column that has seen no row yet
            bf16x8 pf;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float p = pfx_exp2(sv[j] - m_use);
                l_run += p;
                pf[j] = (bf16)p;
            }
            bf16x8 vf[DT];
#pragma unroll
            for (int i = 0; i < DT; ++i) {
                const int d = i * 16 + r;
                vf[i] = *reinterpret_cast<const bf16x8*>(vs + d * PFX_PAIR + (((odd * 4 + c) ^ swz_v(d)) << 3));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < DT; ++i) oacc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i], pf, oacc[i], 0, 0, 0);
        }
        if (odd) vslot = vslot == 2 ? 0 : vslot + 1;
        if (HD == 128)
            kslot = (kslot + 1) & 3;
        else
            kslot = vslot;
    }
    pfx_barrier<0>();   // the loads past the item's end have left before the LDS is given back
    l_run = over_rows<false>(l_run);
    if (active && col < ncols) {
        // record: HD values, and (max, sum) in an array of their own behind all the values.  oacc[i][e]: output element 16 i + 4 c + e
        const int64_t rec = (int64_t)kvh * total_recs + it.rec0 + col;
#pragma unroll
        for (int i = 0; i < DT; ++i) *reinterpret_cast<floatx4*>(records + rec * HD + i * 16 + 4 * c) = oacc[i];
        if (c == 0) *reinterpret_cast<float2*>(records + (int64_t)Hkv * total_recs * HD + rec * 2) = float2{m_run, l_run};
    }
}

// Merges the records of one (worker, head): the items on the worker's list.  Tail
// chunks the step has not reached yet carry weight zero and are never read (nobody
// wrote them).  256 threads: HD / 2 threads span a record, 512 / HD records are read
// side by side, 16 loads in flight per thread (4: 30.6 us at 24 workers, 16: 24.5 us); all sums run in a fixed order.
#define PFX_MAX_ITEMS 1280   // a prefix and a tail of 1024 pieces of 256 rows, up to 256 of them in halves
#define PFX_CT 256
#define PFX_FLIGHT 16
template <int HD>
__global__ __launch_bounds__(PFX_CT) void attn_decode_prefix_combine_kernel(const BlockMeta* __restrict__ tail_meta,
                                                                            const PrefixItem* __restrict__ items,
                                                                            const int32_t* __restrict__ wl_off,
                                                                            const int32_t* __restrict__ wl, int step,
                                                                            const float* __restrict__ records, int64_t total_recs,
                                                                            bf16* __restrict__ o, int Hq, int Hkv) {
    constexpr int TPR = HD / 2;          // threads per record (two floats each)
    constexpr int NS = PFX_CT / TPR;     // records read side by side
    __shared__ float wgt[PFX_MAX_ITEMS];
    __shared__ int32_t roff[PFX_MAX_ITEMS];
    __shared__ float red[PFX_CT / 64];
    __shared__ float2 part[NS][TPR];
    const int b = blockIdx.y, head = blockIdx.x, t = threadIdx.x;
    const int G = Hq / Hkv, kvh = head / G, g = head % G;
    const int tail_rows = tail_meta[b].len + step + 1;
    const int l0 = wl_off[b], n = wl_off[b + 1] - l0;
    const float* val = records + (size_t)kvh * total_recs * HD;                                             // [record][HD]
    const float2* ml = reinterpret_cast<const float2*>(records + (size_t)Hkv * total_recs * HD) + (size_t)kvh * total_recs;   // (max, sum)
    // record index of every item on the list, -1 for a tail chunk not reached yet; running maximum
    float mm = -INFINITY;
    for (int i = t; i < n; i += PFX_CT) {
        const PrefixItem it = items[wl[l0 + i]];
        const bool dead = it.tail && it.row0 >= tail_rows;
        const int ro = dead ? -1 : it.rec0 + (b - it.w0) * G + g;
        roff[i] = ro;
        if (!dead) mm = fmaxf(mm, ml[ro].x);
    }
#pragma unroll
    for (int ofs = 32; ofs > 0; ofs >>= 1) mm = fmaxf(mm, __shfl_xor(mm, ofs, 64));
    if ((t & 63) == 0) red[t >> 6] = mm;
    __syncthreads();
    mm = red[0];
#pragma unroll
    for (int i = 1; i < PFX_CT / 64; ++i) mm = fmaxf(mm, red[i]);
    __syncthreads();   // red[] is reused below
    float l = 0.f;
    for (int i = t; i < n; i += PFX_CT) {
        float wi = 0.f;
        if (roff[i] >= 0) {
            const float2 rec = ml[roff[i]];
            wi = rec.y > 0.f ? pfx_exp2(rec.x - mm) : 0.f;
            l += wi * rec.y;
        }
        wgt[i] = wi;
    }
#pragma unroll
    for (int ofs = 32; ofs > 0; ofs >>= 1) l += __shfl_xor(l, ofs, 64);
    if ((t & 63) == 0) red[t >> 6] = l;
    __syncthreads();   // wgt[] complete as well
    l = red[0];
#pragma unroll
    for (int i = 1; i < PFX_CT / 64; ++i) l += red[i];
    const int sl = t / TPR, e = t % TPR;
    // PFX_FLIGHT records in flight per thread; a record that carries no weight (a tail chunk nobody wrote)
    // is read from a valid address and dropped
    float2 acc = float2{0.f, 0.f};
    for (int i0 = sl; i0 < n; i0 += PFX_FLIGHT * NS) {
        float2 v[PFX_FLIGHT];
        float wi[PFX_FLIGHT];
#pragma unroll
        for (int u = 0; u < PFX_FLIGHT; ++u) {
            const int i = i0 + u * NS;
            wi[u] = i < n ? wgt[i] : 0.f;
            const int ro = i < n ? max(roff[i], 0) : 0;
            v[u] = *reinterpret_cast<const float2*>(val + (size_t)ro * HD + 2 * e);
        }
#pragma unroll
        for (int u = 0; u < PFX_FLIGHT; ++u)
            if (wi[u] != 0.f) {
                acc.x += wi[u] * v[u].x;
                acc.y += wi[u] * v[u].y;
            }
    }
    part[sl][e] = acc;
    __syncthreads();
    if (sl == 0) {
#pragma unroll
        for (int j = 1; j < NS; ++j) {
            acc.x += part[j][e].x;
            acc.y += part[j][e].y;
        }
        bf16x2 out;
        out[0] = (bf16)(acc.x / l);
        out[1] = (bf16)(acc.y / l);
        *reinterpret_cast<bf16x2*>(o + ((size_t)b * Hq + head) * HD + 2 * e) = out;
    }
}

int launch_attn_decode_prefix_bf16(compact_ctx* ctx, const BlockMeta* d_tail_meta, const BlockMeta& shared,
                                   const PrefixItem* d_items, int n_items, const int32_t* d_wl_off, const int32_t* d_wl,
                                   int max_list, int n_workers, int step, const bf16* q, const bf16* kshared,
                                   const bf16* vshared, const bf16* ktail, const bf16* vtail, float* records,
                                   int64_t total_recs, bf16* o, hipStream_t s) {
    const compact_layer_cfg& c = ctx->cfg;
    if (n_items == 0) return COMPACT_OK;
    if (max_list > PFX_MAX_ITEMS) return set_err(ctx, COMPACT_ECAPACITY, "prefix longer than the prefix-aware combine supports");
    const float scale_log2 = LOG2E / sqrtf((float)c.head_dim);
    dim3 grid(n_items, c.n_kv_heads);
    // V^T and K slots: 80 KB at head_dim 128, 48 KB at 64
    const size_t smem = ((size_t)PFX_VSLOTS * PFX_PAIR + (c.head_dim == 128 ? 4 * PFX_TILE : 3 * PFX_PAIR)) * c.head_dim * sizeof(bf16);
    const void* kern = c.head_dim == 128 ? reinterpret_cast<const void*>(attn_decode_prefix_kernel<128>)
                                         : reinterpret_cast<const void*>(attn_decode_prefix_kernel<64>);
    static bool attr[2] = {false, false};
    if (!attr[c.head_dim == 128]) {
        HIP_TRY(ctx, hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr[c.head_dim == 128] = true;
    }
    dim3 cgrid(c.n_q_heads, n_workers);
    if (c.head_dim == 128) {
        {
            ProfileScope ps(ctx, COMPACT_K_ATTN_DECODE, s);
            attn_decode_prefix_kernel<128><<<grid, PFX_WAVES * 64, smem, s>>>(d_tail_meta, shared, d_items, step, q, kshared, vshared,
                                                                             ktail, vtail, records, total_recs, c.n_q_heads,
                                                                             c.n_kv_heads, scale_log2);
        }
        LAUNCH_CHECK(ctx);
        attn_decode_prefix_combine_kernel<128><<<cgrid, PFX_CT, 0, s>>>(d_tail_meta, d_items, d_wl_off, d_wl, step, records,
                                                                     total_recs, o, c.n_q_heads, c.n_kv_heads);
    } else {
        {
            ProfileScope ps(ctx, COMPACT_K_ATTN_DECODE, s);
            attn_decode_prefix_kernel<64><<<grid, PFX_WAVES * 64, smem, s>>>(d_tail_meta, shared, d_items, step, q, kshared, vshared,
                                                                            ktail, vtail, records, total_recs, c.n_q_heads,
                                                                            c.n_kv_heads, scale_log2);
        }
        LAUNCH_CHECK(ctx);
        attn_decode_prefix_combine_kernel<64><<<cgrid, PFX_CT, 0, s>>>(d_tail_meta, d_items, d_wl_off, d_wl, step, records, total_recs, o,
                                                                   c.n_q_heads, c.n_kv_heads);
    }
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
