// Whole-K output projection of a routed layer's decode step for 17 .. 64 rows (bf16
// storage): the kernel of gemv_stream.hip with MT = 2 .. 4 groups of 16 activation
// rows sharing every weight fragment (one MFMA per group and k-step).
//
// Routed layers need the sums of the kernel for at most 16 rows here: the router
// reads what this projection leaves, and a row whose k-th and (k+1)-th logits are
// nearly equal would change an expert, hence its whole output, when the 17th block
// joins a step.  So the split over K between the wavefronts of a workgroup and the
// order in which their partial tiles are added are those of that kernel.  (Dense
// layers take the 64 x 64 ring GEMM with K split over slices, gemm_bf16.hip: its sums
// differ in the last place, and nothing behind them is a choice.  4096 x 4096 at 64
// rows: 19 us here, 12 us there.)
//
//  * the activation rows do not fit in LDS beside the stream (64 rows x K), so they
//    pass through it slice by slice: all wavefronts of the workgroup copy the next
//    slice of K (all rows, whole 128-byte lines, from L2) while the current one
//    feeds the MFMAs, two LDS buffers, one barrier per slice that leaves global
//    loads in flight;
//  * the weight fragments travel through a ring of loads per wavefront, every load
//    unconditional (past the end the last k-step is read again), so that the ring
//    stays in flight across the barriers.
#include <algorithm>

#include "common.h"

#define MTS_WAVES 16

// Workgroup barrier that waits for this wavefront's LDS operations only (global loads stay in flight).
__device__ __forceinline__ void mts_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
}

// A slice of SLICE k of all MT*16 activation rows, runs of 32 that lie 64 apart, copied by NT threads: chunk q (16 bytes)
// of the slice = row q / (SLICE/8), piece q % (SLICE/8); rows past M are zero.
template <int MT, int SLICE, int NT>
struct SliceStager {
    static constexpr int CPR = SLICE / 8;                 // 16-byte pieces per row
    static constexpr int TOTAL = MT * 16 * CPR;           // pieces of a slice
    static constexpr int PER = (TOTAL + NT - 1) / NT;     // pieces per thread (the last round may be partial)
    static constexpr int LDX = SLICE + 8;                 // LDS row stride (elements), padded against bank conflicts
    bf16x8 v[PER];
    __device__ __forceinline__ void load(const bf16* __restrict__ X, int M, int K, int k0, int t) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = min(t + i * NT, TOTAL - 1), row = q / CPR, cc = q % CPR;   // past the end: the last piece again
            v[i] = *reinterpret_cast<const bf16x8*>(X + (size_t)min(row, M - 1) * K + k0 + (cc >> 2) * 64 + (cc & 3) * 8);   // unconditional
        }
    }
    __device__ __forceinline__ void store(bf16* xs, int M, int t) const {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = t + i * NT, row = q / CPR, cc = q % CPR;
            if (TOTAL % NT != 0 && q >= TOTAL) continue;
            bf16x8 w = v[i];
            if (row >= M) {
#pragma unroll
                for (int j = 0; j < 8; ++j) w[j] = (bf16)0.f;
            }
            *reinterpret_cast<bf16x8*>(xs + row * LDX + cc * 8) = w;
        }
    }
};

// ---------------------------------------------------------------------------
// One 16-column tile per workgroup of 16 wavefronts, wavefront kw takes the 64-wide pieces kw, kw + 16, ... of K, a half
// (k-step) at a time: the j-th k-steps of all wavefronts are the j-th slice of 512 k.
// h = resid + X W^T (fp32), hg = bf16(h * g), ssq_parts[tile][m] = sum over the tile's columns of h^2: the output
// projection with the residual add and the front half of the next RMSNorm.
// ---------------------------------------------------------------------------
#define MTS_RING 8
template <int MT>
__global__ __launch_bounds__(MTS_WAVES * 64) void stream_tile_mt_kernel(const bf16* __restrict__ X, const bf16* __restrict__ W,
                                                                        const bf16* __restrict__ resid, const bf16* __restrict__ g,
                                                                        float* __restrict__ h_out, bf16* __restrict__ out16,
                                                                        float* __restrict__ ssq_parts, int M, int N, int K) {
    typedef SliceStager<MT, 512, MTS_WAVES * 64> Stager;
    constexpr int LDX = Stager::LDX;
    extern __shared__ __attribute__((aligned(16))) char smem_mt[];
    bf16* xs0 = reinterpret_cast<bf16*>(smem_mt);                 // two slices [MT*16][LDX] ...
    bf16* xs1 = xs0 + MT * 16 * LDX;
    floatx4(*red)[MTS_WAVES * 64] = reinterpret_cast<floatx4(*)[MTS_WAVES * 64]>(smem_mt);   // ... reused for the partial tiles
    const int t = threadIdx.x, lane = t & 63;
    const int kw = __builtin_amdgcn_readfirstlane(t >> 6);
    const int r = lane & 15, c = lane >> 4;
    const int tile = blockIdx.x;
    const int S = K / 512;   // slices = k-steps per wavefront
    const bf16* w0 = W + (size_t)(tile * 16 + r) * K + c * 8;
    // k-steps 2 i and 2 i + 1 of a wavefront are the halves of one 64-wide piece
    auto first = [](int j) { return (j >> 1) * 1024 + (j & 1) * 32; };   // of wavefront 0
    auto wk = [&](int j) { return first(j) + kw * 64; };
    bf16x8 wf[MTS_RING];
#pragma unroll
    for (int i = 0; i < MTS_RING; ++i) wf[i] = *reinterpret_cast<const bf16x8*>(w0 + wk(min(i, S - 1)));
    Stager st;
    st.load(X, M, K, first(0), t);
    st.store(xs0, M, t);
    st.load(X, M, K, first(1), t);
    mts_barrier();
    floatx4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < S; j0 += MTS_RING) {
#pragma unroll
        for (int i = 0; i < MTS_RING; ++i) {
            const int j = j0 + i;
            if (j < S) {   // uniform
                const bf16* xs = (i & 1) ? xs1 : xs0;   // MTS_RING is even: slice j sits in buffer j & 1 = i & 1
                bf16* xn = (i & 1) ? xs0 : xs1;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(xs + (mt * 16 + r) * LDX + kw * 32 + c * 8);
                    acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], b, acc[mt], 0, 0, 0);
                }
                wf[i] = *reinterpret_cast<const bf16x8*>(w0 + wk(min(j + MTS_RING, S - 1)));
                // slice j + 1 (loaded one round ago) goes into the buffer round j - 1 has finished with
                st.store(xn, M, t);
                st.load(X, M, K, first(min(j + 2, S - 1)), t);
                mts_barrier();
            }
        }
    }
    // (the last round's barrier has passed: nobody reads the slices any more)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) red[mt][kw * 64 + lane] = acc[mt];
    __syncthreads();
    if (kw >= MT) return;
    // wavefront kw finishes group kw: the 16 partial tiles in wavefront order
    const int mt = kw;
    floatx4 v = red[mt][lane];
#pragma unroll
    for (int w = 1; w < MTS_WAVES; ++w) {
        const floatx4 o = red[mt][w * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += o[e];
    }
    // v[e]: activation row m = mt*16 + r, output column n = tile*16 + 4c + e
    const int m = mt * 16 + r;
    float ss = 0.f;
    if (m < M) {
        const size_t o = (size_t)m * N + tile * 16 + 4 * c;
        const bf16x4 rv = *reinterpret_cast<const bf16x4*>(resid + o);
        const bf16x4 gv = *reinterpret_cast<const bf16x4*>(g + tile * 16 + 4 * c);
        bf16x4 hg;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] += (float)rv[e];
            hg[e] = (bf16)(v[e] * (float)gv[e]);
            ss += v[e] * v[e];
        }
        *reinterpret_cast<floatx4*>(h_out + o) = v;
        *reinterpret_cast<bf16x4*>(out16 + o) = hg;
    }
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (c == 0 && m < M) ssq_parts[(size_t)tile * M + m] = ss;
}

bool stream_mt_supported(int M, int N, int K) { return M > 16 && M <= 64 && N % 16 == 0 && K >= 1024 && K % 1024 == 0; }

template <int MT>
static int launch_tile_cfg(compact_ctx* ctx, const bf16* X, const bf16* W, const bf16* resid, const bf16* g, float* h_out,
                           bf16* out16, float* ssq_parts, int M, int N, int K, hipStream_t s) {
    // two activation slices, reused for the MT x 16 KB of partial tiles at the end
    const size_t smem = std::max((size_t)2 * MT * 16 * (512 + 8) * sizeof(bf16), (size_t)MT * MTS_WAVES * 64 * sizeof(floatx4));
    static bool attr = false;
    if (!attr) {
        HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(stream_tile_mt_kernel<MT>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr = true;
    }
    stream_tile_mt_kernel<MT><<<N / 16, MTS_WAVES * 64, smem, s>>>(X, W, resid, g, h_out, out16, ssq_parts, M, N, K);
    LAUNCH_CHECK(ctx);
    return COMPACT_OK;
}

int launch_resid_norm_stream_mt(compact_ctx* ctx, const bf16* X, const bf16* W, const bf16* resid, const bf16* g, float* h_out,
                                bf16* hg_out, float* ssq_parts, int M, int N, int K, hipStream_t s) {
    if (!stream_mt_supported(M, N, K)) return set_err(ctx, COMPACT_ESHAPE, "whole-K streaming kernel for 17..64 rows does not cover this shape");
    switch ((M + 15) / 16) {
        case 2: return launch_tile_cfg<2>(ctx, X, W, resid, g, h_out, hg_out, ssq_parts, M, N, K, s);
        case 3: return launch_tile_cfg<3>(ctx, X, W, resid, g, h_out, hg_out, ssq_parts, M, N, K, s);
        default: return launch_tile_cfg<4>(ctx, X, W, resid, g, h_out, hg_out, ssq_parts, M, N, K, s);
    }
}
