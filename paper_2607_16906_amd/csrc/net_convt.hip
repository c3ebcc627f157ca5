// 2x2 stride-2 transposed convolution and its data gradient with streamed weights (BF16 and FP32).
//
// Forward: a GEMM per input pixel with M = 4 parities x output channels and K = input channels;
// data gradient: M = input channels and K = 4 parities x output channels. A block of WM x WP wavefronts
// owns 16 PB WP consecutive pixels of the whole batch (no rows, hence no padding at their ends) and
// 16 MB WM rows of M. The pixels' K values go through LDS in stages of KS operands of 64 bytes;
// the weights come from memory straight into registers, packed in the order of their use, PF
// operands ahead (see net_stream.h).
//
// Bound by the bytes it writes (four outputs per input pixel) where the grid fills the GPU, by the
// chain of loads of one block where it does not. The staged kernels ran one row segment of at most 64
// pixels per block, with the weights behind the same barriers. Measured, BF16, staged -> streamed:
// forward 512 -> 256 channels at 68^2 34 -> 14 us, 256 -> 128 at 64 x 20^2 75 -> 23 us, 256 -> 128 at 37^2
// 8.2 -> 5.2 us; data gradient of 64 x 20^2 101 -> 24 us. FP32 256 -> 128 at 32 x 12^2 76 -> 20 us.
#include "net_stream.h"

namespace hz {

template <class S, int PB, int MB, int WM, int WP, int PF, bool DG>
__device__ __forceinline__ void convT2s_tile(const typename S::P::T* __restrict__ x, int KC,
                                             const void* __restrict__ wf, const float* __restrict__ bias,
                                             typename S::P::T* __restrict__ y, int MC,
                                             const typename S::P::T* __restrict__ mask, int W, int64_t npix,
                                             int mgrp, int64_t px0, int skipped) {
    using P = typename S::P;
    using T = typename P::T;
    constexpr int CK = P::CK;
    constexpr int PX = 16 * PB * WP, NT = 64 * WM * WP;
    constexpr int KS = 512 / PX < 16 ? 512 / PX : 16;      // operands per stage
    constexpr int NV = PX * KS * 4 / NT;                    // 16-byte vectors of a stage per thread (at most)
    constexpr int RB = KS * 64 + 16;                        // LDS bytes per pixel
    static_assert(NT == 256 && NV * NT == PX * KS * 4 && (KS & (KS - 1)) == 0 && KS % PF == 0, "stage layout");
    __shared__ __attribute__((aligned(16))) unsigned char xl[PX * RB];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv % WM, wp = wv / WM;
    const int lr = lane & 15, lg = lane >> 4;
    const int nk = (DG ? 4 : 1) * KC / CK;   // operands in all

    // a stage's vectors per pixel: those of KS operands, or of all of them where they are fewer (and a
    // power of two)
    const int vpx = 4 * (nk < KS && (nk & (nk - 1)) == 0 ? nk : KS);
    const int ppi = NT / vpx, nv = PX / ppi;   // pixels per pass, passes
    const int part = threadIdx.x & (vpx - 1), pxt = threadIdx.x / vpx;
    // first source pixel of vector i's pixel (data gradient: its parity 0 of the fine grid)
    int64_t src[NV];
    uint32_t ok = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (i >= nv) break;
        const int64_t q = px0 + pxt + i * ppi;
        const bool in = q < npix;
        const int64_t qq = in ? q : 0;
        ok |= (in ? 1u : 0u) << i;
        if (DG) {
            // row iy of sample bz is row bz H + iy of the batch, and 2 (bz H + iy) of its fine grid
            const uint32_t row = (uint32_t)qq / (uint32_t)W, ix = (uint32_t)qq - row * W;
            src[i] = (int64_t)(2 * row) * (2 * W) + 2 * ix;
        } else {
            src[i] = qq;
        }
    }
    uint4 rx[NV];
    auto gload = [&](int s0) {
        const int ks = min(s0 + part / 4, nk - 1);   // (past the last operand: loaded, never used)
        int64_t dp = 0;
        int ch = ks;
        if (DG) {
            dp = (int64_t)((ks & 3) >> 1) * 2 * W + (ks & 1);
            ch = ks >> 2;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (i < nv)
                rx[i] = *(const uint4*)((const unsigned char*)(x + (src[i] + dp) * KC + ch * CK) + (part & 3) * 16);
    };
    auto lstore = [&]() {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (i >= nv) break;
            const uint4 v = ((ok >> i) & 1u) ? rx[i] : uint4{0, 0, 0, 0};
            unsigned char* dst = xl + (pxt + i * ppi) * RB;
            if constexpr (S::STEPS == 1) {
                *(uint4*)(dst + part * 16) = v;
            } else {   // channel 4 q + j of the 16 at position 4 j + q (StF32)
                uint32_t* d = (uint32_t*)(dst + (part / 4) * 64) + (part & 3);
                d[0] = v.x;
                d[4] = v.y;
                d[8] = v.z;
                d[12] = v.w;
            }
        }
    };
    const int mb0 = (mgrp * WM + wm) * MB;
    const unsigned char* wa = (const unsigned char*)wf + (int64_t)mb0 * nk * 1024 + lane * 16;
    uint4 a[PF][MB];
    auto aload = [&](int slot, int ks) {
#pragma unroll
        for (int m = 0; m < MB; ++m) a[slot][m] = *(const uint4*)(wa + ((int64_t)m * nk + ks) * 1024);
    };
    f32x4_t acc[PB][MB];
#pragma unroll
    for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[p][m] = f32x4_t{0, 0, 0, 0};
    gload(0);
#pragma unroll
    for (int t = 0; t < PF; ++t) aload(t, t);
    asm volatile("" ::: "memory");   // keep the loads above the test
    if (skipped) return;             // uniform over the block
    const unsigned char* xb = xl + (wp * PB * 16 + lr) * RB + lg * 16;
    for (int s0 = 0; s0 < nk; s0 += KS) {
        if (s0) __syncthreads();
        lstore();
        __syncthreads();
        if (s0 + KS < nk) gload(s0 + KS);
        const int s1 = min(nk, s0 + KS);
        for (int k0 = s0; k0 < s1; k0 += PF) {
            uint4 b[PF][PB];
#pragma unroll
            for (int t = 0; t < PF; ++t)
#pragma unroll
                for (int p = 0; p < PB; ++p) b[t][p] = *(const uint4*)(xb + p * 16 * RB + (k0 - s0 + t) * 64);
            if constexpr (DG && S::STEPS > 1) {
                // the staged kernel's order: step by step, the 4 parities within a step
#pragma unroll
                for (int u = 0; u < PF; u += 4)
#pragma unroll
                    for (int st = 0; st < S::STEPS; ++st)
#pragma unroll
                        for (int t = u; t < u + 4; ++t)
#pragma unroll
                            for (int p = 0; p < PB; ++p)
#pragma unroll
                                for (int m = 0; m < MB; ++m) acc[p][m] = S::mma(a[t][m], b[t][p], acc[p][m], st);
#pragma unroll
                for (int t = 0; t < PF; ++t) aload(t, min(k0 + PF + t, nk - 1));
            } else {
#pragma unroll
                for (int t = 0; t < PF; ++t) {
#pragma unroll
                    for (int st = 0; st < S::STEPS; ++st)
#pragma unroll
                        for (int p = 0; p < PB; ++p)
#pragma unroll
                            for (int m = 0; m < MB; ++m) acc[p][m] = S::mma(a[t][m], b[t][p], acc[p][m], st);
                    aload(t, min(k0 + PF + t, nk - 1));
                }
            }
        }
    }
    // register r of a lane holds row 16 (mb0 + m) + 4 lg + r of M for pixel px0 + 16 (wp PB + p) + lr
    const int ncob = MC / 16;
    float bv[MB][4];
    if (!DG) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) bv[m][r] = bias[((mb0 + m) >> 1) % ncob * 16 + 4 * lg + r];
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
        const int64_t q = px0 + (wp * PB + p) * 16 + lr;
        if (q >= npix) continue;
        if (DG) {
            T mk[MB][4];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const T* ms = mask + q * MC + (mb0 + m) * 16 + 4 * lg;
                if constexpr (sizeof(T) == 2) *(uint2*)mk[m] = *(const uint2*)ms;
                else *(uint4*)mk[m] = *(const uint4*)ms;
            }
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                float t[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) t[r] = P::val(mk[m][r]) > 0.0f ? acc[p][m][r] : 0.0f;
                P::store4(y + q * MC + (mb0 + m) * 16 + 4 * lg, t);
            }
        } else {
            // row block mb of M: (parity a, 16-channel block, parity b), b fastest
            const uint32_t row = (uint32_t)q / (uint32_t)W, ix = (uint32_t)q - row * W;
            T* yq = y + ((int64_t)(2 * row) * (2 * W) + 2 * ix) * MC + 4 * lg;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const int mb = mb0 + m;
                const int pa = mb / (2 * ncob), cob = (mb >> 1) - pa * ncob, pb = mb & 1;
                float t[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) t[r] = acc[p][m][r] + bv[m][r];
                P::store4(yq + (int64_t)(pa * 2 * W + pb) * MC + cob * 16, t);
            }
        }
    }
}

// grid: x = (pixel tile, M group), M group fastest
template <class S, int PB, int MB, int WM, int WP, int PF, bool DG>
__global__ __launch_bounds__(256, 2) void k_convT2s(const typename S::P::T* __restrict__ x, int KC,
                                                    const void* __restrict__ wf, const float* __restrict__ bias,
                                                    typename S::P::T* __restrict__ y, int MC,
                                                    const typename S::P::T* __restrict__ mask, int W,
                                                    int64_t npix, int ngrp, const int* __restrict__ skip) {
    const int skipped = skip ? *skip : 0;
    const int v = xcd_linear(blockIdx.x, gridDim.x);
    const int grp = v % ngrp;
    convT2s_tile<S, PB, MB, WM, WP, PF, DG>(x, KC, wf, bias, y, MC, mask, W, npix, grp,
                                            (int64_t)(v / ngrp) * (16 * PB * WP), skipped);
}

// Ragged batch: job = (system, M group, pixel tile) in (sys, c0, ty0).
template <class S, int PB, int MB, int WM, int WP, int PF>
__global__ __launch_bounds__(256, 2) void k_convT2s_jobs(const TileJob* __restrict__ jobs,
                                                         const LayerIO* __restrict__ io, const void* __restrict__ wf,
                                                         const float* __restrict__ bias, int cin_p, int cout_p) {
    using T = typename S::P::T;
    const TileJob jb = jobs[xcd_linear(blockIdx.x, gridDim.x)];
    const LayerIO d = io[jb.sys];
    if (d.stop && *d.stop) return;
    convT2s_tile<S, PB, MB, WM, WP, PF, false>((const T*)d.x0, cin_p, wf, bias, (T*)d.y, cout_p, nullptr, d.W,
                                               (int64_t)d.H * d.W, jb.c0, (int64_t)jb.ty0 * (16 * PB * WP), 0);
}

template <class S, int PB, int MB, int WM, int WP, bool DG>
static int launch_pf(const ConvT2sArgs<typename S::P>& g, int ngrp, hipStream_t s) {
    constexpr int PX = 16 * PB * WP;
    const int64_t nblk = (g.npix + PX - 1) / PX * ngrp;
    if (nblk > INT32_MAX || g.npix > INT32_MAX) {
        set_error("convT2: grid too large");
        return HZ_ERR_ARG;
    }
    const int nk = (DG ? 4 : 1) * g.KC / S::P::CK;
#define HZ_CT(F)                                                                                                    \
    do {                                                                                                            \
        if (g.jobs) {                                                                                               \
            if constexpr (!DG)                                                                                      \
                hipLaunchKernelGGL((k_convT2s_jobs<S, PB, MB, WM, WP, F>), dim3(g.njobs), dim3(256), 0, s, g.jobs,  \
                                   g.io, g.wf, g.bias, g.KC, g.MC);                                                 \
        } else {                                                                                                    \
            hipLaunchKernelGGL((k_convT2s<S, PB, MB, WM, WP, F, DG>), dim3((unsigned)nblk), dim3(256), 0, s, g.x, g.KC, \
                               g.wf, g.bias, g.y, g.MC, g.mask, g.W, g.npix, ngrp, g.skip);                    \
        }                                                                                                           \
    } while (0)
    if constexpr (PB * MB <= 4) {   // short blocks: more operands in flight
        if (nk % 8 == 0) HZ_CT(8);
        else if (nk % 4 == 0) HZ_CT(4);
        else if constexpr (!DG) HZ_CT(2);
    } else {
        if (nk % 4 == 0) HZ_CT(4);
        else if constexpr (!DG) HZ_CT(2);
    }
#undef HZ_CT
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

template <class S>
static int launch_any(int form, const ConvT2sArgs<typename S::P>& g, bool dgrad, hipStream_t s) {
    const ConvT2sForm f = convT2s_form(form);
    const int mblk = dgrad ? g.MC / 16 : g.MC / 4;
    if (f.px == 0 || !convT2s_layer_ok<typename S::P>(g.KC, g.MC, dgrad) || mblk % f.mblk || !g.wf) {
        set_error("convT2: the streamed form does not take these channels");
        return HZ_ERR_ARG;
    }
    const int ngrp = mblk / f.mblk;
    switch (form) {
#define HZ_CT(ID, PB, MB, WM, WP)                                              \
    case ID:                                                                   \
        if (dgrad) return launch_pf<S, PB, MB, WM, WP, true>(g, ngrp, s);      \
        return launch_pf<S, PB, MB, WM, WP, false>(g, ngrp, s);
        HZ_CONVT2S_FORMS(HZ_CT)
#undef HZ_CT
    }
    return HZ_ERR_ARG;
}

template <>
int launch_convT2s<PolBF16>(int form, const ConvT2sArgs<PolBF16>& g, bool dgrad, hipStream_t s) {
    return launch_any<StBF16>(form, g, dgrad, s);
}
template <>
int launch_convT2s<PolF32>(int form, const ConvT2sArgs<PolF32>& g, bool dgrad, hipStream_t s) {
    return launch_any<StF32>(form, g, dgrad, s);
}

}  // namespace hz
