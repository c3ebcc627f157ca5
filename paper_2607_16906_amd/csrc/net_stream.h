// 3x3 convolution with streamed weights: device code shared by the BF16 and FP32 launchers.
//
// A block of WC x WR wavefronts owns a (RPW WR) x 16 pixel tile and 16 NCB WC output channels;
// wavefront (wc, wr) computes rows [RPW wr, RPW (wr + 1)) of 16 NCB channels. Only the input patch
// goes through LDS. The weights come from memory straight into registers, packed in the order in
// which a wavefront feeds them to the matrix cores (conv3s_index: one 1 KB line per 16 x 32
// operand), PF taps ahead of their use, so that no weight is staged, waited for at a barrier or
// read back from LDS.
//
// Why: with weights in LDS a wavefront of 2 rows x 32 channels reads 30 operands from LDS for 36
// matrix instructions, more than the LDS delivers (128 bytes per clock per CU against one 1 KB
// operand pair per 16 clocks on each of 4 SIMDs). Here the same LDS feeds RPW rows of pixels to
// NCB channel blocks: (RPW + 2) 3 reads for 9 RPW NCB instructions.
//
// Measured (BF16, best staged form -> streamed): 512 -> 256 channels at 136^2 64 -> 44 us (983 TFLOP/s), 64 ->
// 64 at 544^2 52 -> 35 us, 256 -> 128 at 64 x 40^2 98 -> 60 us, 256 -> 256 at 37^2 11.0 -> 7.8 us. FP32: 256 -> 128
// at 32 x 24^2 139 -> 115 us (95 of 157 TFLOP/s, with a quarter of the 16-pixel columns outside the image).
// What is left is latency: on large grids the matrix cores are busy for 31 to 38 % of the cycles and the LDS
// for 20 to 25 %, with 2 to 3 wavefronts per SIMD that wait at one barrier per chunk; on small grids a block's
// chain of chunks.
#pragma once

#include "net_kernels.h"

namespace hz {

// One operand is 16 bytes per lane: 8 BF16 channels (one 16x16x32 instruction), or 4 FP32 channels
// lg, 4 + lg, 8 + lg, 12 + lg of a 16-channel chunk (four 16x16x4 instructions, which take channels
// 4 s .. 4 s + 3 in step s as conv3_chunk_mma does).
struct StBF16 {
    using P = PolBF16;
    __device__ static f32x4_t mma(uint4 a, uint4 b, f32x4_t c, int) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                       c, 0, 0, 0);
    }
    static constexpr int STEPS = 1;
};
struct StF32 {
    using P = PolF32;
    __device__ static f32x4_t mma(uint4 a, uint4 b, f32x4_t c, int s) {
        const f32x4_t x = __builtin_bit_cast(f32x4_t, a), y = __builtin_bit_cast(f32x4_t, b);
        return __builtin_amdgcn_mfma_f32_16x16x4f32(x[s], y[s], c, 0, 0, 0);
    }
    static constexpr int STEPS = 4;
};

constexpr int CS_PB = 80;   // bytes per patch pixel in LDS (one chunk is 64 B; + 16 B against bank conflicts)

enum { CS_PLAIN = 0, CS_POOL = 1, CS_MASKED = 2, CS_HEAD = 3 };

// One tile. x0, x1, y, ypool and ex's tensors point at the sample. Every output is accumulated chunk
// by chunk, tap by tap in row-major order, with the operands and order of conv3_chunk_mma (the same
// result bits as the staged forms).
template <class S, int NCB, int RPW, int WC, int WR, int EPI>
__device__ __forceinline__ void conv3s_tile(const typename S::P::T* __restrict__ x0, int c0,
                                            const typename S::P::T* __restrict__ x1, int c1,
                                            const void* __restrict__ wf, const float* __restrict__ bias,
                                            typename S::P::T* __restrict__ y, int cout_p,
                                            typename S::P::T* __restrict__ ypool, int H, int W, int relu,
                                            const Conv3Out& ex, int co0, int ty0, int tx0, int skipped) {
    using P = typename S::P;
    using T = typename P::T;
    constexpr int CK = P::CK;                               // channels per chunk: 64 bytes of a pixel
    constexpr int VE = 16 / (int)sizeof(T);
    constexpr int NT = 64 * WC * WR, TH = RPW * WR;
    constexpr int NPX = (TH + 2) * 18;
    constexpr int NU = NPX * 4, NPT = (NU + NT - 1) / NT;   // 16-byte vectors of a chunk, per thread
    constexpr int PSZ = NPX * CS_PB;
    constexpr int PF = NCB == 1 && RPW <= 4 ? 9 : 3;        // taps of weights in flight
    static_assert(CK * sizeof(T) == 64, "a chunk is 64 bytes of a pixel");
    static_assert(EPI != CS_HEAD || WC == 1, "the fused head needs every channel in one wavefront");
    static_assert(EPI != CS_POOL || RPW % 2 == 0, "pooling needs row pairs in one wavefront");
    __shared__ __attribute__((aligned(16))) unsigned char patch[2 * PSZ];   // double-buffered

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wc = wv % WC, wr = wv / WC;
    const int lr = lane & 15, lg = lane >> 4;
    const int nch = (c0 + c1) / CK;
    const int ncob = cout_p / 16;

    // staging: vector i of this thread belongs to patch pixel px; pix: its image pixel (0 where it lies
    // outside: loaded all the same, stored as zeros)
    int pix[NPT];
    uint32_t ok = 0;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int u = min((int)threadIdx.x + i * NT, NU - 1);
        const int px = u >> 2;
        const int py = px / 18, pxx = px - py * 18;
        const int gy = ty0 + py - 1, gx = tx0 + pxx - 1;
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
        pix[i] = in ? gy * W + gx : 0;
        ok |= (in ? 1u : 0u) << i;
    }
    const int q4 = threadIdx.x & 3;   // NT is a multiple of 4: the same quarter of the chunk every time
    uint4 ra[NPT];
    auto gload = [&](int kc) {
        const int k0 = kc * CK;
        const bool first = k0 < c0;
        const T* src = (first ? x0 + k0 : x1 + (k0 - c0)) + q4 * VE;
        const int cc = first ? c0 : c1;
#pragma unroll
        for (int i = 0; i < NPT; ++i) ra[i] = *(const uint4*)(src + (int64_t)pix[i] * cc);
    };
    auto lstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
            const int u = (int)threadIdx.x + i * NT;
            if (u < NU) {
                const uint4 v = ((ok >> i) & 1u) ? ra[i] : uint4{0, 0, 0, 0};
                unsigned char* dst = patch + buf * PSZ + (u >> 2) * CS_PB;
                if constexpr (S::STEPS == 1) {
                    *(uint4*)(dst + q4 * 16) = v;
                } else {   // channel 4 q + j of the chunk at position 4 j + q: step q of lane group j
                    uint32_t* d = (uint32_t*)dst + q4;
                    d[0] = v.x;
                    d[4] = v.y;
                    d[8] = v.z;
                    d[12] = v.w;
                }
            }
        }
    };
    // weight operands: [chunk][channel block][tap][lane][16 B]
    const unsigned char* wb = (const unsigned char*)wf + (int64_t)(co0 / 16 + wc * NCB) * (9 * 1024) + lane * 16;
    const int64_t wch = (int64_t)ncob * (9 * 1024);
    uint4 a[PF][NCB];
    auto aload = [&](int slot, const unsigned char* wk, int tap) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) a[slot][cb] = *(const uint4*)(wk + (cb * 9 + tap) * 1024);
    };
    f32x4_t acc[RPW][NCB];
#pragma unroll
    for (int r = 0; r < RPW; ++r)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = f32x4_t{0, 0, 0, 0};
    gload(0);
#pragma unroll
    for (int t = 0; t < PF; ++t) aload(t, wb, t);
    asm volatile("" ::: "memory");   // keep the loads above the test
    if (skipped) return;             // uniform over the block

    for (int kc = 0; kc < nch; ++kc) {
        // one barrier per chunk: the buffer written here was last read two chunks ago, before the
        // previous chunk's barrier
        const int buf = kc & 1;
        lstore(buf);
        __syncthreads();
        if (kc + 1 < nch) gload(kc + 1);
        const unsigned char* wk = wb + kc * wch;
        const unsigned char* wn = kc + 1 < nch ? wk + wch : wk;   // (past the last chunk: reloaded, unused)
        const unsigned char* pb = patch + buf * PSZ + ((wr * RPW) * 18 + lr) * CS_PB + lg * 16;
        auto bload = [&](int row, int dx) { return *(const uint4*)(pb + (row * 18 + dx) * CS_PB); };
        uint4 b[RPW + 2][3];
#pragma unroll
        for (int r = 0; r < RPW; ++r) b[r][0] = bload(r, 0);
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3, dx = tap % 3;
            if (tap + 1 < 9) {   // the next tap's new rows
                const int ny = (tap + 1) / 3, nx = (tap + 1) % 3;
                if (ny == 0) {
#pragma unroll
                    for (int r = 0; r < RPW; ++r) b[r][nx] = bload(r, nx);
                } else {
                    b[RPW + ny - 1][nx] = bload(RPW + ny - 1, nx);
                }
            }
#pragma unroll
            for (int st = 0; st < S::STEPS; ++st)
#pragma unroll
                for (int r = 0; r < RPW; ++r)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
                        acc[r][cb] = S::mma(a[tap % PF][cb], b[r + dy][dx], acc[r][cb], st);
            const int nt = tap + PF;
            aload(tap % PF, nt < 9 ? wk : wn, nt % 9);
            __builtin_amdgcn_sched_barrier(0);   // keeps the loads that far ahead of their use
        }
    }

    // epilogue: register r of a lane holds channel cw + 16 cb + 4 lg + r of pixel (gy0 + row, gx)
    const int cw = co0 + wc * NCB * 16;
    const int gx = tx0 + lr, gy0 = ty0 + wr * RPW;
    if constexpr (EPI == CS_HEAD) {   // 1x1 head over all channels, as conv3_tile's
        float o0[RPW], o1[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) o0[r] = o1[r] = 0.0f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int co = cb * 16 + 4 * lg + q;
                const float w0 = P::val(((const T*)ex.head_w)[co]), w1 = P::val(((const T*)ex.head_w)[cout_p + co]);
                const float bc = bias[co];
#pragma unroll
                for (int r = 0; r < RPW; ++r) {
                    float t = acc[r][cb][q] + bc;
                    if (relu) t = t > 0.0f ? t : 0.0f;
                    t = P::val(P::cvt(t));
                    o0[r] += t * w0;
                    o1[r] += t * w1;
                }
            }
        const float hb0 = ((const float*)ex.head_b)[0], hb1 = ((const float*)ex.head_b)[1];
        const double sfac = ex.head_fixed_s > 0 ? ex.head_fixed_s : ex.head_sc[0];
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            float a0 = o0[r], a1 = o1[r];
            a0 += __shfl_xor(a0, 16, 64);
            a1 += __shfl_xor(a1, 16, 64);
            a0 += __shfl_xor(a0, 32, 64);
            a1 += __shfl_xor(a1, 32, 64);
            const int gy = gy0 + r;
            if (lg == 0 && gy < ex.head_nyt && gx < ex.head_nxt) {
                const double2 zv{sfac * (double)(hb0 + a0), sfac * (double)(hb1 + a1)};
                const int64_t zi = (int64_t)gy * ex.head_nxt + gx;
                if (ex.head_c128) ((double2*)ex.head_z)[zi] = zv;
                else ((float2*)ex.head_z)[zi] = from_d2<float2>(zv);
            }
        }
        return;
    }
    // MASKED: channels below ex.split go to y (ex.split per pixel), the others to ex.y1_; an entry
    // whose mask entry is <= 0 is zero
    const int split = EPI == CS_MASKED && ex.split > 0 ? ex.split : cout_p;
    const bool second = EPI == CS_MASKED && cw >= split;
    const int cst = second ? cout_p - split : split;
    T* yo = (second ? (T*)ex.y1_ : y) + (second ? cw - split : cw) + 4 * lg;
    const T* mo = nullptr;
    if (EPI == CS_MASKED) {
        mo = (const T*)(second ? ex.mask1_ : ex.mask0_);
        if (mo) mo += (second ? cw - split : cw) + 4 * lg;
    }
    float bv[NCB][4];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[cb][q] = bias ? bias[cw + cb * 16 + 4 * lg + q] : 0.0f;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        T mk[RPW][4];
        if (EPI == CS_MASKED && mo) {
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const int gy = gy0 + r;
                if (gy < H && gx < W) {
                    const T* m = mo + ((int64_t)gy * W + gx) * cst + cb * 16;
                    if constexpr (sizeof(T) == 2) *(uint2*)mk[r] = *(const uint2*)m;
                    else *(uint4*)mk[r] = *(const uint4*)m;
                }
            }
        }
        float v[RPW][4];
#pragma unroll
        for (int r = 0; r < RPW; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float t = acc[r][cb][q] + bv[cb][q];
                if (relu) t = t > 0.0f ? t : 0.0f;
                v[r][q] = t;
            }
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int gy = gy0 + r;
            if (gy < H && gx < W) {
                float t[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    t[q] = v[r][q];
                    if (EPI == CS_MASKED && mo && !(P::val(mk[r][q]) > 0.0f)) t[q] = 0.0f;
                }
                P::store4(yo + ((int64_t)gy * W + gx) * cst + cb * 16, t);
            }
        }
        if constexpr (EPI == CS_POOL) {
#pragma unroll
            for (int r = 0; r < RPW; r += 2) {
                float av[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float s = v[r][q] + v[r + 1][q];
                    s += __shfl_xor(s, 1, 64);
                    av[q] = 0.25f * s;
                }
                const int gy = gy0 + r;
                if ((lr & 1) == 0 && gy < H && gx < W)
                    P::store4(ypool + ((int64_t)(gy / 2) * (W / 2) + gx / 2) * cout_p + cw + cb * 16 + 4 * lg, av);
            }
        }
    }
}

// grid: x = blocks; logical order: channel block fastest, then column tile, row tile, sample
template <class S, int NCB, int RPW, int WC, int WR, int EPI>
__global__ __launch_bounds__(64 * WC * WR, 2) void k_conv3s(
    const typename S::P::T* __restrict__ x0, int c0, const typename S::P::T* __restrict__ x1, int c1,
    const void* __restrict__ wf, const float* __restrict__ bias, typename S::P::T* __restrict__ y, int cout_p,
    typename S::P::T* __restrict__ ypool, int H, int W, int relu, const int* __restrict__ skip, Conv3Out ex) {
    using T = typename S::P::T;
    const int skipped = skip ? *skip : 0;
    constexpr int TN = 16 * NCB * WC, TH = RPW * WR;
    const int ncb = cout_p / TN, ntx = (W + 15) / 16, nty = (H + TH - 1) / TH;
    int v = xcd_linear(blockIdx.x, gridDim.x);
    const int cbi = v % ncb;
    v /= ncb;
    const int txi = v % ntx;
    v /= ntx;
    const int tyi = v % nty;
    const int64_t bz = v / nty;
    const int64_t plane = (int64_t)H * W;
    const int s0 = EPI == CS_MASKED && ex.split > 0 ? ex.split : cout_p;
    if (EPI == CS_MASKED) {
        if (ex.y1_) ex.y1_ = (T*)ex.y1_ + bz * plane * (cout_p - s0);
        if (ex.mask0_) ex.mask0_ = (const T*)ex.mask0_ + bz * plane * s0;
        if (ex.mask1_) ex.mask1_ = (const T*)ex.mask1_ + bz * plane * (cout_p - s0);
    }
    conv3s_tile<S, NCB, RPW, WC, WR, EPI>(x0 + bz * plane * c0, c0, x1 ? x1 + bz * plane * c1 : nullptr, c1, wf, bias,
                                          EPI == CS_HEAD ? nullptr : y + bz * plane * s0, cout_p,
                                          EPI == CS_POOL ? ypool + bz * (plane / 4) * cout_p : nullptr, H, W, relu, ex,
                                          cbi * TN, tyi * TH, txi * 16, skipped);
}

// Ragged batch: block b runs job jobs[b] with the system's tensors; with the fused head, column col
// of the system's z.
template <class S, int NCB, int RPW, int WC, int WR, int EPI>
__global__ __launch_bounds__(64 * WC * WR, 2) void k_conv3s_jobs(
    const TileJob* __restrict__ jobs, const LayerIO* __restrict__ io, const void* __restrict__ wf,
    const float* __restrict__ bias, int c0, int c1, int cout_p, const typename S::P::T* __restrict__ head_w,
    const float* __restrict__ head_b, int col, int c128) {
    using T = typename S::P::T;
    const TileJob jb = jobs[xcd_linear(blockIdx.x, gridDim.x)];
    const LayerIO d = io[jb.sys];
    if (d.stop && *d.stop) return;
    Conv3Out ex;
    if constexpr (EPI == CS_HEAD) {
        ex.head_w = head_w;
        ex.head_b = head_b;
        ex.head_c128 = c128;
        ex.head_z = c128 ? (void*)((double2*)d.z + (int64_t)col * d.zld) : (void*)((float2*)d.z + (int64_t)col * d.zld);
        ex.head_nxt = d.nxt;
        ex.head_nyt = d.nyt;
        ex.head_sc = d.sc;
    }
    conv3s_tile<S, NCB, RPW, WC, WR, EPI>((const T*)d.x0, c0, (const T*)d.x1, c1, wf, bias, (T*)d.y, cout_p,
                                          (T*)d.ypool, d.H, d.W, 1, ex, jb.c0, jb.ty0, jb.tx0, 0);
}

}  // namespace hz
