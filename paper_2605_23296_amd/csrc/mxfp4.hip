// Block-scaled 4-bit expert weights (the format the paper's largest model is
// served in, Sec. IV-B "mxfp4 weights"; OCP Microscaling Formats v1.0): FP4
// E2M1 elements, two per byte (even index in the low nibble), one E8M0 scale
// 2^(e-127) per block of 32 consecutive elements along the contraction index.
//
// Routed decode rows are bound by the bytes of the expert weights they stream,
// so reading 4.25 bits per weight instead of 16 is worth 3.76x.  Every product
// of an element and a scale is exact in bf16, so the weights are expanded in
// registers and fed to the same bf16 MFMA as the 16-bit path:
//
//  * a lane loads 16 bytes = one whole block of 32 elements of one weight row;
//    the four lane groups of an MFMA row take four consecutive blocks, so a
//    wave-instruction still reads 64 contiguous bytes of each of 16 rows;
//  * the scale bytes of a slice go through LDS, 32 contiguous bytes of each of
//    16 rows in one load.  A load costs the address path a clock per group of four
//    lanes that is not one contiguous run, whatever it brings: a byte per lane and
//    block, the scales cost as much as the codes (16 rows of the 120B-shaped layer: a
//    step 241 -> 229 us, gate/up + down 119 of it).  The codes through LDS as well,
//    two whole rows per load: half the workgroups per compute unit, 257 us a step;
//  * expansion is the hardware's scaled conversion (v_cvt_scalef32_pk_bf16_fp4:
//    one byte = two elements -> two bf16, times a float scale), so a block of
//    32 costs 16 conversions and the elements come out in their natural order.
#include "common.h"
#include "stream_lds.h"
#include "vecio.h"

#define MX_BLOCK 32
#define MX_KSLICE 1024                       // k per workgroup: 8 blocks per lane in flight
#define MX_GROUPS (MX_KSLICE / (4 * MX_BLOCK))
#define MX_WAVE_BYTES (16 * MX_KSLICE / MX_BLOCK)   // a wavefront's scales in LDS

int mxfp4_ksplit(int K) { return (K + MX_KSLICE - 1) / MX_KSLICE; }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// 2^(e-127) as a float (e in 1..254)
__device__ __forceinline__ float e8m0_to_float(uint32_t scale_byte) { return __uint_as_float(scale_byte << 23); }

// Eight codes (one dword, element i in nibble i) -> eight bf16, each times `scale`.
__device__ __forceinline__ bf16x8 fp4_expand8(uint32_t w, float scale) {
    union {
        bf16x2_t p[4];
        bf16x8 v;
    } out;
#if defined(__HIP_DEVICE_COMPILE__)
    out.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 0);
    out.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 1);
    out.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 2);
    out.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(w, scale, 3);
#else
    (void)w;
    (void)scale;
#endif
    return out.v;
}

// ---------------------------------------------------------------------------
// Expansion to bf16 [rows, K] (the 16-bit copy the prefill GEMMs read).
// One thread per block of 32 elements.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void mxfp4_dequant_kernel(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                                            bf16* __restrict__ out, int64_t n_blocks) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_blocks) return;
    const uint4 cw = *reinterpret_cast<const uint4*>(codes + i * 16);
    const float sc = e8m0_to_float(scales[i]);
    const uint32_t w[4] = {cw.x, cw.y, cw.z, cw.w};
#pragma unroll
    for (int d = 0; d < 4; ++d) *reinterpret_cast<bf16x8*>(out + i * MX_BLOCK + d * 8) = fp4_expand8(w[d], sc);
}

int launch_mxfp4_dequant(compact_ctx* ctx, const uint8_t* codes, const uint8_t* scales, bf16* out, int64_t rows, int K,
                         hipStream_t s) {
    if (rows < 0 || K < MX_BLOCK || K % MX_BLOCK != 0) return set_err(ctx, COMPACT_ESHAPE, "4-bit weights need K % 32 == 0");
    const int64_t nb = rows * (K / MX_BLOCK);
    if (nb == 0) return COMPACT_OK;
    mxfp4_dequant_kernel<<<(unsigned)((nb + 255) / 256), 256, 0, s>>>(codes, scales, out, nb);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

// ---------------------------------------------------------------------------
// Per-expert weight streaming for routed decode rows, 4-bit weights:
// partials[slice][sorted row][N] = X[rows of expert e, kslice] W_e[N, kslice]^T.
// One workgroup per k-slice, 64 weight rows and expert tile; 4 wavefronts of 16 weight rows each.  X, like the scales, lands in
// LDS directly, its source rows looked up before the weights are asked for (16 x 8192, a step: 252 -> 247 us when only the rows
// that are there were staged).  A row's codes are K / 2 and its scales K / 32 bytes, so the slices share 128-byte lines (K 2880:
// 512 of 1440 bytes touch five lines, and the scales of all three slices lie in the same ones): the slices of the same rows run
// on one XCD (slice_item), whose L2 asks for a line once.  Bound by HBM: gate/up + down of 16 rows of the 120B-shaped layer
// (640 MB) 120 -> 113 us, a step 228 -> 221; d 1600, F 1088, 64 experts, 16 rows 88 -> 84; K a multiple of 256 as before.  Four
// neighbouring lanes on 64 bytes of a row gain nothing (56.5 and 57.6 us a launch), 8 or 16 wavefronts a workgroup lose (60 -> 61, 64.5).
// ---------------------------------------------------------------------------
struct MxGroup {
    const int32_t* expert_list;  // [n_tiles] experts to run, -1 = none (null: tile e = expert e)
    const int32_t* tile_row0;    // [n_tiles] first sorted row of the tile (null: the expert's first row)
    const int32_t* tile_rows;    // [n_tiles] its rows, at most 16 (null: all of the expert's rows)
    const int32_t* offsets;    // [E + 1] rows of every expert in the expert-sorted order
    const int32_t* a_gather;   // [total_rows] source row of X, or null (X already sorted)
    int64_t q_expert_stride;   // bytes between consecutive experts' codes
    int64_t s_expert_stride;   // bytes between consecutive experts' scales
    int total_rows;
    int n_tiles;               // entries of the list, or experts
};

__global__ __launch_bounds__(256) void gemm_skinny_mxfp4_kernel(const bf16* __restrict__ X, const uint8_t* __restrict__ Wq,
                                                                const uint8_t* __restrict__ Ws, float* __restrict__ P, int N,
                                                                int K, const MxGroup grp) {
    constexpr int LDX = MX_KSLICE + 8;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16* xs = reinterpret_cast<bf16*>(smem);  // [16][LDX]
    const int lane = threadIdx.x & 63, wave = wave_index();
    const int r = lane & 15, c = lane >> 4;
    const SliceItem it = slice_item(blockIdx.x, (K + MX_KSLICE - 1) / MX_KSLICE, (N + 63) / 64);
    const int slice = it.slice, y = it.col, z = it.tile;
    if (z >= grp.n_tiles) return;
    const int e = grp.expert_list ? grp.expert_list[z] : z;
    if (e < 0) return;
    const int row_base = grp.tile_row0 ? grp.tile_row0[z] : grp.offsets[e];
    const int M = min(grp.tile_rows ? grp.tile_rows[z] : grp.offsets[e + 1] - row_base, 16);
    if (M <= 0) return;   // nobody was routed to this expert
    Wq += (size_t)e * grp.q_expert_stride;
    Ws += (size_t)e * grp.s_expert_stride;
    const int k0 = slice * MX_KSLICE;
    const int klen = min(MX_KSLICE, K - k0);
    const int nblk = klen / MX_BLOCK;            // blocks of this slice
    const int n0 = (y * 4 + wave) * 16;
    const bool active = n0 < N;
    uint8_t* const scales = reinterpret_cast<uint8_t*>(smem) + 16 * LDX * sizeof(bf16) + wave * MX_WAVE_BYTES;   // [16 rows][32]

    int src[4];   // rows of X that this wavefront stages
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        src[i] = row_base + min(wave + 4 * i, M - 1);
        if (grp.a_gather) src[i] = grp.a_gather[src[i]];
    }
    // the weight stream goes first: everything below overlaps with it.  Past the row's end: its last block again.
    uint4 cw[MX_GROUPS];
    if (active) {
        const uint8_t* wp = Wq + (size_t)(n0 + r) * (K / 2) + k0 / 2;
#pragma unroll
        for (int g = 0; g < MX_GROUPS; ++g) cw[g] = *reinterpret_cast<const uint4*>(wp + min(4 * g + c, nblk - 1) * 16);
    }
    // Activations of this expert's rows, a wavefront per row, past the row's end its last piece again.  An expert seldom has
    // more than two or three rows: the MFMA columns beyond them repeat the last row (nobody reads their sums).
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (wave + 4 * i < M) {
            const bf16* xp = X + (size_t)src[i] * K + k0;
#pragma unroll
            for (int j = 0; j < MX_KSLICE / 512; ++j)
                load16_to_lds(xp + min(j * 64 + lane, klen / 8 - 1) * 8, xs + (wave + 4 * i) * LDX + j * 512);
        }
    // Scale bytes: four lanes a row, eight bytes each (rows are K / 32 bytes, so any alignment); a short row's pieces overlap.
    if (active) {
        const uint8_t* sp = Ws + (size_t)(n0 + (lane >> 2)) * (K / MX_BLOCK) + k0 / MX_BLOCK;
        uint8_t* const dst = scales + (lane >> 2) * 32;
        if (nblk >= 8) {
            const int at = min((lane & 3) * 8, nblk - 8);
            uint64_t v;
            __builtin_memcpy(&v, sp + at, 8);
            __builtin_memcpy(dst + at, &v, 8);
        } else {
#pragma unroll 1
            for (int j = lane & 3; j < nblk; j += 4) dst[j] = sp[j];
        }
    }
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0);   // what was loaded into LDS has landed
#endif
    __syncthreads();
    if (!active) return;

    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    const bf16* xrow = xs + min(r, M - 1) * LDX + c * MX_BLOCK;
    auto group = [&](int g, bool whole) {
        const int blk = 4 * g + c;
        const bool there = whole || blk < nblk;   // a block past the row's end contributes nothing
        const uint32_t sb = scales[r * 32 + blk];
        const float scale = e8m0_to_float(there ? sb : 127u);
        const uint32_t w[4] = {cw[g].x, cw[g].y, cw[g].z, cw[g].w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            bf16x8 b = *reinterpret_cast<const bf16x8*>(xrow + g * 4 * MX_BLOCK + d * 8);
            if (!there) {
#pragma unroll
                for (int j = 0; j < 8; ++j) b[j] = (bf16)0.f;
            }
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp4_expand8(there ? w[d] : 0u, scale), b, acc, 0, 0, 0);
        }
    };
    if (nblk == MX_KSLICE / MX_BLOCK) {
#pragma unroll
        for (int g = 0; g < MX_GROUPS; ++g) group(g, true);
    } else {
#pragma unroll
        for (int g = 0; g < MX_GROUPS; ++g)
            if (4 * g < nblk) group(g, false);
    }
    // acc[e]: activation row r, weight row n0 + 4c + e
    if (r < M) *reinterpret_cast<floatx4*>(P + ((size_t)slice * grp.total_rows + row_base + r) * N + n0 + 4 * c) = acc;
}

int launch_gemm_skinny_grouped_mxfp4(compact_ctx* ctx, const bf16* X, const int32_t* a_gather, const uint8_t* Wq,
                                     const uint8_t* Ws, const int32_t* offsets, int n_experts, int total_rows,
                                     float* partials, int N, int K, int ks, hipStream_t s, const int32_t* expert_list,
                                     int n_listed, const int32_t* tile_row0, const int32_t* tile_rows) {
    if (N % 16 != 0 || K % MX_BLOCK != 0) return set_err(ctx, COMPACT_ESHAPE, "4-bit weight streaming needs N % 16 == 0 and K % 32 == 0");
    if (ks != mxfp4_ksplit(K)) return set_err(ctx, COMPACT_EINVAL, "unexpected K split");
    const int n_tiles = expert_list ? n_listed : n_experts;
    MxGroup g{expert_list, tile_row0, tile_rows, offsets, a_gather, (int64_t)N * (K / 2), (int64_t)N * (K / MX_BLOCK), total_rows, n_tiles};
    const int64_t grid = slice_items(ks, (N + 63) / 64, n_tiles);
    if (grid >= 1 << 24) return set_err(ctx, COMPACT_ESHAPE, "too many workgroups for 4-bit weight streaming");
    constexpr int smem = 16 * (MX_KSLICE + 8) * (int)sizeof(bf16) + 4 * MX_WAVE_BYTES;
    gemm_skinny_mxfp4_kernel<<<(unsigned)grid, 256, smem, s>>>(X, Wq, Ws, partials, N, K, g);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}
