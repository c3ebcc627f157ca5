// Weight gradients on the matrix cores (FP32 accumulation): products with the pixels as the reduction
// index,
//   3x3:            dW[tap][co][ci] = sum_p G[p][co] X[p + tap][ci],   db[co] = sum_p G[p][co]
//   transposed 2x2: dW[ab][co][ci] = sum_i G[2i + ab][co] x[i][ci],    db[co] = sum_p G[p][co]
//
// Both tensors are stored with the channels of a pixel together, the matrix instruction wants a run
// of pixels per channel. A tile is staged as it lies in memory (16-byte loads and LDS stores, 16
// channels of all pixels to a plane) and turned on the way into the registers by the transposing LDS
// read (ds_read_b64_tr_b16: 16 lanes read 4 pixels x 16 channels, each receives the 4 pixels of its
// channel). A pixel offset is then only an address, so the taps share one copy of the input patch.
//
// Reduction step: 32 pixels, 8 consecutive ones per group of 16 lanes. The 4 groups take 4 places of
// the tile (TW / 8 columns of 8, the rest rows apart), and a wavefront walks down R rows: the input
// operands of row q serve the three taps dy at the output rows q, q - 1 and q - 2, so that per step
// 3 input operands and 2 of G are read for 18 products (LDS bandwidth allows two products a read).
//
// The 3x3 kernel sees the batch as one image of B (H + 1) rows, a row of zeros after each sample, and
// tiles its rows with no remainder per sample; TW is 8 or 16 by the width. Blocks of one chunk of
// tiles read the same pixels for different channels: they are given to one XCD, whose L2 then holds
// them. Partials [chunk][tap][co][ci] are summed in a fixed order by k_wgrad_reduce.
//
// Measured (BF16, batch 64): 160^2 pixels 32 -> 32 channels 79 -> 55 us (HBM: 210 MB, 42 us), 64 -> 32 145
// -> 81 us; 80^2 128 -> 64 147 -> 68 us, 40^2 256 -> 128 172 -> 66 us (0.92 PF); transposed 64 -> 32 to 160^2
// 63 -> 35 us, 256 -> 128 to 40^2 76 -> 29 us, against tiles transposed in registers into an LDS copy per
// column offset.
#include <algorithm>

#include "train_wgrad.h"

namespace hz {

namespace {

struct WgBF16 {
    using T = bf16_t;
    static constexpr int PXB = 32;   // bytes of 16 channels of a pixel
    static constexpr int VC = 8;     // channels per 16-byte vector
    using Op = bf16x8_t;             // 8 pixels of the lane's channel
    struct Row {                     // the three column offsets of one row
        Op v[3];
    };
    // lane part of an operand's address; group kg = lane / 16 starts at byte g
    struct Lane {
        const unsigned char *p0, *p1;
    };
    __device__ static Lane lane(const unsigned char* lds, int g) {
        // the two 4-pixel halves of the run, odd groups the other half first (groups are a multiple
        // of 256 bytes apart: this way two of them hit different banks)
        const int l = threadIdx.x & 15, h = (threadIdx.x >> 4) & 1;
        const unsigned char* p = lds + g + (l >> 2) * PXB + (l & 3) * 8;
        return Lane{p + h * 4 * PXB, p + (1 - h) * 4 * PXB};
    }
    __device__ static Op op(const Lane& a, int off) {
        typedef __attribute__((ext_vector_type(4))) short s4;
        typedef __attribute__((address_space(3))) s4* lp;
        struct {
            s4 a, b;
        } r;
        r.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a.p0 + off));
        r.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(a.p1 + off));
        return __builtin_bit_cast(Op, r);
    }
    __device__ static Row row(const Lane& a, int off) {
        return Row{{op(a, off), op(a, off + PXB), op(a, off + 2 * PXB)}};
    }
    __device__ static Op ones() {
        const uint4 u{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
        return __builtin_bit_cast(Op, u);
    }
    __device__ static f32x4_t mma(const Op& a, const Op& b, f32x4_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static f32x4_t mma(const Op& a, const Row& b, int dx, f32x4_t c) { return mma(a, b.v[dx], c); }
};

using S = WgBF16;

// bytes of a plane of n pixels, padded so that the 8 lanes of one LDS store phase (16 bytes each,
// the channels of a pixel, then the next pixel) hit different banks
constexpr int wg_plane(int n, int pxb, int mod) { return (n * pxb + 127) / 128 * 128 + mod; }

// The chunk and channel tile of this block: of 8 consecutive blocks, one per XCD, each takes its own
// chunk, all its channel tiles in turn (chunk counts below 8 would leave XCDs out: plain order there).
__device__ inline void wg_block(int nct, int nchunk, int* z, int* ct) {
    const int id = blockIdx.x;
    if (nchunk >= 8) {
        const int k = id >> 3;
        *z = (k / nct) * 8 + (id & 7);
        *ct = k % nct;
    } else {
        *z = id / nct;
        *ct = id % nct;
    }
}

constexpr f32x4_t WG_ZERO = {0.f, 0.f, 0.f, 0.f};

// Sum the accumulators of the WK wavefronts that share a channel tile into the first one's, through
// the LDS, in order.
template <int WK, int N>
__device__ __forceinline__ void wg_sum(f32x4_t (&acc)[N], unsigned char* lds, int wk, int wtile) {
    if constexpr (WK > 1) {
        f32x4_t* buf = (f32x4_t*)lds + (size_t)wtile * N * 64 + (threadIdx.x & 63);
#pragma unroll 1
        for (int k = 1; k < WK; ++k) {
            __syncthreads();
            if (wk == k) {
#pragma unroll
                for (int i = 0; i < N; ++i) buf[i * 64] = acc[i];
            }
            __syncthreads();
            if (wk == 0) {
#pragma unroll
                for (int i = 0; i < N; ++i) acc[i] += buf[i * 64];
            }
        }
    }
}

// 3x3. Block: 32 WCO output x 16 WCI input channels, a wavefront 32 x 16 of them for all 9 taps (WK
// wavefronts share those and split the rows). Tile: TW columns x 32 R / TW rows.
template <int WCO, int WCI, int WK, int R, int TW>
__global__ __launch_bounds__(64 * WCO * WCI * WK, 2) void k_wgrad3(const WgradArgs<bf16_t> A) {
    constexpr int NT = 64 * WCO * WCI * WK;
    constexpr int GC = TW / 8;                  // lane groups side by side
    constexpr int TH = 4 / GC * R, PW = TW + 2, PH = TH + 2;
    constexpr int CO = 32 * WCO, CI = 16 * WCI, RS = R / WK;
    constexpr int PLG = wg_plane(TW * TH, S::PXB, CO >= 64 ? 32 : 64);
    constexpr int PLX = wg_plane(PW * PH, S::PXB, CI >= 64 ? 32 : 64);
    constexpr int NVG = CO / S::VC, NVX = CI / S::VC;   // vectors per pixel
    constexpr int NG = (TW * TH * NVG + NT - 1) / NT, NX = (PW * PH * NVX + NT - 1) / NT;
    constexpr int LDS = PLG * (CO / 16) + PLX * (CI / 16);
    constexpr int SUM = WK > 1 ? WCO * WCI * 20 * 64 * 16 : 0;
    __shared__ __attribute__((aligned(16))) unsigned char lds[LDS > SUM ? LDS : SUM];
    unsigned char* const ldx = lds + PLG * (CO / 16);

    int z, ct;
    wg_block(A.nct, A.nchunk, &z, &ct);
    if (z >= A.nchunk) return;
    const int nci = (A.cin_p + CI - 1) / CI;
    const int ci0 = (ct % nci) * CI, co0 = (ct / nci) * CO;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int wci = w % WCI, wco = (w / WCI) % WCO, wk = w / (WCI * WCO);
    const int kg = lane >> 4;
    const int H = A.H, W = A.W, Hg = H + 1, rows = A.B * Hg;
    const int tx_n = (W + TW - 1) / TW;

    f32x4_t acc[20];   // [co block][tap], then the bias sums of the two co blocks
#pragma unroll
    for (int i = 0; i < 20; ++i) acc[i] = WG_ZERO;
    const bool bias = ci0 == 0 && wci == 0;

    uint4 rg[NG], rx[NX];
    auto gload = [&](int tile) {
        const int row0 = (tile / tx_n) * TH, tx0 = (tile % tx_n) * TW;
        const int b0 = row0 / Hg, y0 = row0 - b0 * Hg;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT;
            const int c = co0 + (v % NVG) * S::VC, px = v / NVG;
            const int x = tx0 + px % TW;
            int y = y0 + px / TW, b = b0;
            while (y >= Hg) y -= Hg, ++b;
            rg[i] = uint4{0, 0, 0, 0};
            if ((TW * TH * NVG % NT == 0 || v < TW * TH * NVG) && b < A.B && y < H && x < W && c < A.cout_p)
                rg[i] = *(const uint4*)(A.G + (((int64_t)b * H + y) * W + x) * A.cout_p + c);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT;
            const int c = ci0 + (v % NVX) * S::VC, px = v / NVX;
            const int x = tx0 + px % PW - 1;
            int y = y0 + px / PW - 1, b = b0;
            while (y >= Hg) y -= Hg, ++b;
            rx[i] = uint4{0, 0, 0, 0};
            if ((PW * PH * NVX % NT == 0 || v < PW * PH * NVX) && b < A.B && y >= 0 && y < H && x >= 0 && x < W &&
                c < A.cin_p) {
                const int64_t pix = ((int64_t)b * H + y) * W + x;
                rx[i] = *(const uint4*)(c < A.c0 ? A.x0 + pix * A.c0 + c : A.x1 + pix * (A.cin_p - A.c0) + (c - A.c0));
            }
        }
    };
    auto lstore = [&]() {
        constexpr int VP = 16 / S::VC;   // vectors of a plane's pixel
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT, cv = v % NVG, px = v / NVG;
            if (TW * TH * NVG % NT == 0 || v < TW * TH * NVG)
                *(uint4*)(lds + (cv / VP) * PLG + px * S::PXB + (cv % VP) * 16) = rg[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, cv = v % NVX, px = v / NVX;
            if (PW * PH * NVX % NT == 0 || v < PW * PH * NVX)
                *(uint4*)(ldx + (cv / VP) * PLX + px * S::PXB + (cv % VP) * 16) = rx[i];
        }
    };
    // this lane group's place in the tile
    const int gy = (kg / GC) * R + wk * RS, gx = (kg % GC) * 8;
    const S::Lane lg = S::lane(lds + wco * 2 * PLG, (gy * TW + gx) * S::PXB);
    const S::Lane lx = S::lane(ldx + wci * PLX, (gy * PW + gx) * S::PXB);

    const int t_beg = z * A.tpc, t_end = min(((rows + TH - 1) / TH) * tx_n, t_beg + A.tpc);
    if (t_beg < t_end) gload(t_beg);
    for (int tile = t_beg; tile < t_end; ++tile) {
        __syncthreads();   // the previous tile's reads of the LDS are done
        lstore();
        __syncthreads();
        if (tile + 1 < t_end) gload(tile + 1);
        S::Row xr[3];
        xr[0] = S::row(lx, 0);
        xr[1] = S::row(lx, PW * S::PXB);
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            xr[(s + 2) % 3] = S::row(lx, (s + 2) * PW * S::PXB);
            S::Op g[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) g[k] = S::op(lg, s * TW * S::PXB + k * PLG);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        acc[k * 9 + dy * 3 + dx] = S::mma(g[k], xr[(s + dy) % 3], dx, acc[k * 9 + dy * 3 + dx]);
            if (bias) {
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[18 + k] = S::mma(g[k], S::ones(), acc[18 + k]);
            }
        }
    }
    wg_sum<WK>(acc, lds, wk, wco * WCI + wci);
    if (wk) return;
    // lane holds D[co = 4 kg + r][ci = lane % 16] of every block
    const int ci = ci0 + wci * 16 + (lane & 15);
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = co0 + wco * 32 + k * 16 + 4 * kg + r;
            if (co >= A.cout_p) continue;
            if (ci < A.cin_p) {
#pragma unroll
                for (int t = 0; t < 9; ++t)
                    A.part[(((int64_t)z * 9 + t) * A.cout_p + co) * A.cin_p + ci] = acc[k * 9 + t][r];
            }
            if (bias && (lane & 15) == 0) A.partb[(int64_t)z * A.cout_p + co] = acc[18 + k][r];
        }
}

// Transposed 2x2. Block: 32 output x 64 input channels, a wavefront 32 x 32 of them for the 4
// parities; two wavefronts share those and split the rows. Tile: 16 columns x 2 R rows of coarse
// pixels of the batch's B H rows; G is staged by parity, so that a run of coarse pixels is a run there.
template <int R>
__global__ __launch_bounds__(256, 2) void k_wgradT(const WgradArgs<bf16_t> A) {
    constexpr int NT = 256, TW = 16, TH = 2 * R, CO = 32, CI = 64, WK = 2, RS = R / WK, NPX = TW * TH;
    constexpr int PLG = wg_plane(NPX, S::PXB, 32), PLX = PLG;
    constexpr int NVG = CO / S::VC, NVX = CI / S::VC;
    constexpr int NG = 4 * NPX * NVG / NT, NX = NPX * NVX / NT;
    static_assert(4 * NPX * NVG % NT == 0 && NPX * NVX % NT == 0 && RS >= 1, "whole vectors per thread");
    constexpr int LDS = PLG * 8 + PLX * 4;
    constexpr int SUM = 2 * 18 * 64 * 16;
    __shared__ __attribute__((aligned(16))) unsigned char lds[LDS > SUM ? LDS : SUM];
    unsigned char* const ldx = lds + PLG * 8;   // G: plane [parity][16 channels]

    int z, ct;
    wg_block(A.nct, A.nchunk, &z, &ct);
    if (z >= A.nchunk) return;
    const int nci = (A.cin_p + CI - 1) / CI;
    const int ci0 = (ct % nci) * CI, co0 = (ct / nci) * CO;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int wci = w & 1, wk = w >> 1;
    const int kg = lane >> 4;
    const int W = A.W, rows = A.B * A.H;
    const int tx_n = (W + TW - 1) / TW;

    f32x4_t acc[18];   // [ab][co block][ci block], then the bias sums of the two co blocks
#pragma unroll
    for (int i = 0; i < 18; ++i) acc[i] = WG_ZERO;
    const bool bias = ci0 == 0 && wci == 0;

    uint4 rg[NG], rx[NX];
    auto gload = [&](int tile) {
        const int row0 = (tile / tx_n) * TH, tx0 = (tile % tx_n) * TW;
#pragma unroll
        for (int i = 0; i < NG; ++i) {   // fine pixels of the tile, rows of 2 TW
            const int v = threadIdx.x + i * NT;
            const int c = co0 + (v % NVG) * S::VC, px = v / NVG;
            const int x = 2 * tx0 + px % (2 * TW), y = 2 * row0 + px / (2 * TW);
            rg[i] = uint4{0, 0, 0, 0};
            if (y < 2 * rows && x < 2 * W && c < A.cout_p)
                rg[i] = *(const uint4*)(A.G + ((int64_t)y * (2 * W) + x) * A.cout_p + c);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT;
            const int c = ci0 + (v % NVX) * S::VC, px = v / NVX;
            const int x = tx0 + px % TW, y = row0 + px / TW;
            rx[i] = uint4{0, 0, 0, 0};
            if (y < rows && x < W && c < A.cin_p)
                rx[i] = *(const uint4*)(A.x0 + ((int64_t)y * W + x) * A.cin_p + c);
        }
    };
    auto lstore = [&]() {
        constexpr int VP = 16 / S::VC;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT, cv = v % NVG, px = v / NVG;
            const int fx = px % (2 * TW), fy = px / (2 * TW);
            const int pl = ((fy & 1) * 2 + (fx & 1)) * 2 + cv / VP;
            *(uint4*)(lds + pl * PLG + ((fy >> 1) * TW + (fx >> 1)) * S::PXB + (cv % VP) * 16) = rg[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, cv = v % NVX, px = v / NVX;
            *(uint4*)(ldx + (cv / VP) * PLX + px * S::PXB + (cv % VP) * 16) = rx[i];
        }
    };
    const int g = (((kg >> 1) * R + wk * RS) * TW + (kg & 1) * 8) * S::PXB;
    const S::Lane lg = S::lane(lds, g), lx = S::lane(ldx + wci * 2 * PLX, g);

    const int t_beg = z * A.tpc, t_end = min(((rows + TH - 1) / TH) * tx_n, t_beg + A.tpc);
    if (t_beg < t_end) gload(t_beg);
    for (int tile = t_beg; tile < t_end; ++tile) {
        __syncthreads();   // the previous tile's reads of the LDS are done
        lstore();
        __syncthreads();
        if (tile + 1 < t_end) gload(tile + 1);
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const int o = s * TW * S::PXB;
            S::Op xb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) xb[i] = S::op(lx, o + i * PLX);
#pragma unroll
            for (int ab = 0; ab < 4; ++ab)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const S::Op ga = S::op(lg, o + (ab * 2 + k) * PLG);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[(ab * 2 + k) * 2 + i] = S::mma(ga, xb[i], acc[(ab * 2 + k) * 2 + i]);
                    if (bias) acc[16 + k] = S::mma(ga, S::ones(), acc[16 + k]);
                }
        }
    }
    wg_sum<WK>(acc, lds, wk, wci);
    if (wk) return;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = co0 + k * 16 + 4 * kg + r;
            if (co >= A.cout_p) continue;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int ci = ci0 + wci * 32 + i * 16 + (lane & 15);
                if (ci >= A.cin_p) continue;
#pragma unroll
                for (int ab = 0; ab < 4; ++ab)
                    A.part[(((int64_t)z * 4 + ab) * A.cout_p + co) * A.cin_p + ci] = acc[(ab * 2 + k) * 2 + i][r];
            }
            if (bias && (lane & 15) == 0) A.partb[(int64_t)z * A.cout_p + co] = acc[16 + k][r];
        }
}

// ------------------------------------------------------------------ FP32
//
// v_mfma_f32_16x16x4_f32 takes one value per lane, 4 pixels x 16 channels: a read of 256 consecutive
// bytes of the planes above, so nothing is transposed. It adds its 4 products one after the other
// (fma, in the order of k), which makes every sum below a plain chain over the pixels of the chunk.
// The matrix cores are what bounds these (32 clocks for 1 K products; 145 TF measured).

constexpr int WF_PX = 64;   // bytes of 16 channels of a pixel

// 3x3. Block: 32 x 32 channels over its chunk of 8 x 16 pixel tiles of the samples, wavefront w the
// pair (w / 2, w % 2) for all 9 taps; the chain takes a tile's rows in turn and 4 pixels a step. The
// operands of an input row serve 3 output rows from registers.
// Measured, batch 32 at 96^2: 32 -> 32 channels 57 -> 55 us, 64 -> 32 107 -> 104 us (105 TF), against tiles
// transposed in LDS by 4-byte stores; what is left to the 145 TF is whole blocks of an uneven share
// of the CUs. (Four blocks to a CU, 128 registers, spill the loads in flight: 101 and 149 us.)
__global__ __launch_bounds__(256, 3) void k_wgrad3_f32(const WgradArgs<float> A) {
    constexpr int TW = 16, TH = 8, PW = 18, PH = 10, NT = 256;
    constexpr int PLG = TW * TH * WF_PX + 64, PLX = PW * PH * WF_PX + 64;
    constexpr int NG = TW * TH * 8 / NT, NX = (PW * PH * 8 + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * PLG + 2 * PLX];
    unsigned char* const ldx = lds + 2 * PLG;
    int z, ct;
    wg_block(A.nct, A.nchunk, &z, &ct);
    if (z >= A.nchunk) return;
    const int nci = (A.cin_p + 31) / 32;
    const int ci0 = (ct % nci) * 32, co0 = (ct / nci) * 32;
    const int lane = threadIdx.x & 63, lr = lane & 15, kg = lane >> 4, w = threadIdx.x >> 6;
    const int cob = w >> 1, cib = w & 1;
    const int H = A.H, W = A.W;
    const int tx_n = (W + TW - 1) / TW, per_img = tx_n * ((H + TH - 1) / TH);
    f32x4_t acc[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) acc[i] = WG_ZERO;
    const int bco = threadIdx.x & 31, bseg = threadIdx.x >> 5;   // bias: one output channel, one row
    float accb = 0.f;

    float4 rg[NG], rx[NX];
    auto gload = [&](int tile) {
        const int b = tile / per_img, r = tile - b * per_img;
        const int ty0 = (r / tx_n) * TH, tx0 = (r % tx_n) * TW;
        const int64_t p0 = (int64_t)b * H * W;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT, c = co0 + (v & 7) * 4, px = v >> 3;
            const int y = ty0 + px / TW, x = tx0 + px % TW;
            rg[i] = float4{0.f, 0.f, 0.f, 0.f};
            if (y < H && x < W && c < A.cout_p)
                rg[i] = *(const float4*)(A.G + (p0 + (int64_t)y * W + x) * A.cout_p + c);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, c = ci0 + (v & 7) * 4, px = v >> 3;
            const int y = ty0 + px / PW - 1, x = tx0 + px % PW - 1;
            rx[i] = float4{0.f, 0.f, 0.f, 0.f};
            if (v < PW * PH * 8 && y >= 0 && y < H && x >= 0 && x < W && c < A.cin_p) {
                const int64_t pix = p0 + (int64_t)y * W + x;
                rx[i] = *(const float4*)(c < A.c0 ? A.x0 + pix * A.c0 + c : A.x1 + pix * (A.cin_p - A.c0) + (c - A.c0));
            }
        }
    };
    auto lstore = [&]() {
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT, cv = v & 7, px = v >> 3;
            *(float4*)(lds + (cv >> 2) * PLG + px * WF_PX + (cv & 3) * 16) = rg[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, cv = v & 7, px = v >> 3;
            if (v < PW * PH * 8) *(float4*)(ldx + (cv >> 2) * PLX + px * WF_PX + (cv & 3) * 16) = rx[i];
        }
    };
    const unsigned char* const lg = lds + cob * PLG + kg * WF_PX + lr * 4;
    const unsigned char* const lx = ldx + cib * PLX + kg * WF_PX + lr * 4;
    const unsigned char* const lb = lds + (bco >> 4) * PLG + bseg * TW * WF_PX + (bco & 15) * 4;
    const int t_beg = z * A.tpc, t_end = min(per_img * A.B, t_beg + A.tpc);
    if (t_beg < t_end) gload(t_beg);
    for (int tile = t_beg; tile < t_end; ++tile) {
        __syncthreads();   // the previous tile's reads of the LDS are done
        lstore();
        __syncthreads();
        if (tile + 1 < t_end) gload(tile + 1);
        if (ci0 == 0) {
#pragma unroll
            for (int k = 0; k < TW; ++k) accb += *(const float*)(lb + k * WF_PX);
        }
        float xr[3][3][4];   // [row][dx][4 pixels]
        auto row = [&](int r) {
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int q = 0; q < 4; ++q) xr[r % 3][dx][q] = *(const float*)(lx + (r * PW + 4 * q + dx) * WF_PX);
        };
        float g[2][4];       // of this row and the next
        auto grow = [&](int r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) g[r & 1][q] = *(const float*)(lg + (r * TW + 4 * q) * WF_PX);
        };
        row(0);
        row(1);
        grow(0);
#pragma unroll
        for (int r = 0; r < TH; ++r) {
            row(r + 2);      // (used last: its reads take the time of the first two rows' products)
            if (r + 1 < TH) grow(r + 1);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int t = 6 * h; t < 6 + 3 * h; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(g[r & 1][q], xr[(r + t / 3) % 3][t % 3][q], acc[t],
                                                                      0, 0, 0);
        }
    }
    // lane holds D[co = 4 kg + r][ci = lr]
    const int ci = ci0 + cib * 16 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int co = co0 + cob * 16 + 4 * kg + r;
        if (ci >= A.cin_p || co >= A.cout_p) continue;
#pragma unroll
        for (int t = 0; t < 9; ++t) A.part[(((int64_t)z * 9 + t) * A.cout_p + co) * A.cin_p + ci] = acc[t][r];
    }
    if (ci0 == 0) {   // the rows' sums, pairwise
        float* red = (float*)lds;
        __syncthreads();
        red[bseg * 32 + bco] = accb;
        __syncthreads();
        if (threadIdx.x < 32 && co0 + bco < A.cout_p) {
            float s[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] = red[k * 32 + bco];
            A.partb[(int64_t)z * A.cout_p + co0 + bco] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
        }
    }
}

// Transposed 2x2. Block: 16 output x 32 input channels over its chunk of 8 x 8 coarse tiles of the
// samples, wavefront ab the parity ab: one operand of G and two of x for two products. G is staged by
// parity. Measured, batch 32: 64 -> 32 channels to 96^2 200 -> 39 us, 256 -> 128 to 24^2 104 -> 35 us, against one
// thread per channel pair without the matrix cores.
__global__ __launch_bounds__(256, 4) void k_wgradT_f32(const WgradArgs<float> A) {
    constexpr int NPX = 64, NT = 256, PL = NPX * WF_PX + 64;
    constexpr int NG = 4 * NPX * 4 / NT, NX = NPX * 8 / NT;
    __shared__ __attribute__((aligned(16))) unsigned char lds[6 * PL];   // G [parity], x [16 channels]
    unsigned char* const ldx = lds + 4 * PL;
    int z, ct;
    wg_block(A.nct, A.nchunk, &z, &ct);
    if (z >= A.nchunk) return;
    const int nci = (A.cin_p + 31) / 32;
    const int ci0 = (ct % nci) * 32, co0 = (ct / nci) * 16;
    const int lane = threadIdx.x & 63, lr = lane & 15, kg = lane >> 4, ab = threadIdx.x >> 6;
    const int H = A.H, W = A.W;
    const int tx_n = (W + 7) / 8, per_img = tx_n * ((H + 7) / 8);
    f32x4_t acc[2] = {WG_ZERO, WG_ZERO}, accb = WG_ZERO;
    const bool bias = ci0 == 0 && ab == 0;

    float4 rg[NG], rx[NX];
    auto gload = [&](int tile) {
        const int b = tile / per_img, r = tile - b * per_img;
        const int ty0 = (r / tx_n) * 8, tx0 = (r % tx_n) * 8;
#pragma unroll
        for (int i = 0; i < NG; ++i) {   // fine pixels of the tile, rows of 16
            const int v = threadIdx.x + i * NT, c = co0 + (v & 3) * 4, px = v >> 2;
            const int y = 2 * ty0 + px / 16, x = 2 * tx0 + px % 16;
            rg[i] = float4{0.f, 0.f, 0.f, 0.f};
            if (y < 2 * H && x < 2 * W)
                rg[i] = *(const float4*)(A.G + (((int64_t)b * 2 * H + y) * (2 * W) + x) * A.cout_p + c);
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, c = ci0 + (v & 7) * 4, px = v >> 3;
            const int y = ty0 + px / 8, x = tx0 + px % 8;
            rx[i] = float4{0.f, 0.f, 0.f, 0.f};
            if (y < H && x < W && c < A.cin_p)
                rx[i] = *(const float4*)(A.x0 + (((int64_t)b * H + y) * W + x) * A.cin_p + c);
        }
    };
    auto lstore = [&]() {
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const int v = threadIdx.x + i * NT, px = v >> 2, fx = px % 16, fy = px / 16;
            *(float4*)(lds + ((fy & 1) * 2 + (fx & 1)) * PL + ((fy >> 1) * 8 + (fx >> 1)) * WF_PX + (v & 3) * 16) = rg[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int v = threadIdx.x + i * NT, cv = v & 7, px = v >> 3;
            *(float4*)(ldx + (cv >> 2) * PL + px * WF_PX + (cv & 3) * 16) = rx[i];
        }
    };
    const int lo = kg * WF_PX + lr * 4;
    const int t_beg = z * A.tpc, t_end = min(per_img * A.B, t_beg + A.tpc);
    if (t_beg < t_end) gload(t_beg);
    for (int tile = t_beg; tile < t_end; ++tile) {
        __syncthreads();   // the previous tile's reads of the LDS are done
        lstore();
        __syncthreads();
        if (tile + 1 < t_end) gload(tile + 1);
#pragma unroll
        for (int q = 0; q < NPX / 4; ++q) {
            const int o = lo + 4 * q * WF_PX;
            const float g = *(const float*)(lds + ab * PL + o);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(g, *(const float*)(ldx + i * PL + o), acc[i], 0, 0, 0);
            if (bias) {   // the 4 parities of a coarse pixel, then the chain over those
                const float s = ((g + *(const float*)(lds + PL + o)) + *(const float*)(lds + 2 * PL + o)) +
                                *(const float*)(lds + 3 * PL + o);
                accb = __builtin_amdgcn_mfma_f32_16x16x4f32(s, 1.f, accb, 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int co = co0 + 4 * kg + r;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ci = ci0 + i * 16 + lr;
            if (ci < A.cin_p) A.part[(((int64_t)z * 4 + ab) * A.cout_p + co) * A.cin_p + ci] = acc[i][r];
        }
        if (bias && lr == 0) A.partb[(int64_t)z * A.cout_p + co] = accb[r];
    }
}

// chunks of ntiles tiles over nct channel tiles: 512 blocks (two per CU) where the tiles allow it, at
// most cap chunks
template <class T>
void wg_chunks(WgradArgs<T>& a, int ntiles, int nct, int cap) {
    int want = std::max(1, 512 / nct);
    if (want > 8) want = want / 8 * 8;
    want = std::min(std::min(want, cap), ntiles);
    a.nct = nct;
    a.tpc = (ntiles + want - 1) / want;
    a.nchunk = (ntiles + a.tpc - 1) / a.tpc;
}

template <class T>
unsigned wg_grid(const WgradArgs<T>& a) {
    return (unsigned)((a.nchunk >= 8 ? (a.nchunk + 7) / 8 * 8 : a.nchunk) * a.nct);
}

template <int WCO, int WCI, int WK, int TW>
int run3(WgradArgs<bf16_t>& a, int cap, hipStream_t s) {
    constexpr int R = 8, TH = 32 * R / TW;
    const int ntiles = (a.B * (a.H + 1) + TH - 1) / TH * ((a.W + TW - 1) / TW);
    wg_chunks(a, ntiles, (a.cin_p + 16 * WCI - 1) / (16 * WCI) * ((a.cout_p + 32 * WCO - 1) / (32 * WCO)), cap);
    hipLaunchKernelGGL((k_wgrad3<WCO, WCI, WK, R, TW>), dim3(wg_grid(a)), dim3(64 * WCO * WCI * WK), 0, s, a);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

template <int WCO, int WCI, int WK>
int run3w(WgradArgs<bf16_t>& a, int cap, hipStream_t s) {
    // 8 columns where 16 would cover more of nothing (W = 20: 24 columns, not 32)
    return (a.W + 15) / 16 * 2 > (a.W + 7) / 8 ? run3<WCO, WCI, WK, 8>(a, cap, s)
                                               : run3<WCO, WCI, WK, 16>(a, cap, s);
}

}  // namespace

int launch_wgrad3(WgradArgs<bf16_t>& a, int cap, hipStream_t s) {
    // the channel tile: 32 x 64 where the layer has them (both tensors are staged once per channel
    // tile of the other), 32 x 32, or 32 x 16 for the few channels of the first layer
    if (a.cin_p <= 16) return run3w<1, 1, 4>(a, cap, s);
    if (a.cin_p % 64 == 0) return run3w<1, 4, 1>(a, cap, s);
    if (a.cout_p % 64 == 0) return run3w<2, 2, 1>(a, cap, s);
    return run3w<1, 2, 2>(a, cap, s);
}

int launch_wgradT(WgradArgs<bf16_t>& a, int cap, hipStream_t s) {
    constexpr int R = 4, TH = 2 * R;
    const int ntiles = (a.B * a.H + TH - 1) / TH * ((a.W + 15) / 16);
    wg_chunks(a, ntiles, (a.cin_p + 63) / 64 * ((a.cout_p + 31) / 32), cap);
    hipLaunchKernelGGL((k_wgradT<R>), dim3(wg_grid(a)), dim3(256), 0, s, a);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_wgrad3(WgradArgs<float>& a, int cap, hipStream_t s) {
    // about 1024 blocks, as many chunks as the partial buffer holds
    const int ntiles = (a.W + 15) / 16 * ((a.H + 7) / 8) * a.B;
    a.nct = (a.cin_p + 31) / 32 * ((a.cout_p + 31) / 32);
    const int want = std::min(std::min(512, (1024 + a.nct - 1) / a.nct), cap);
    a.tpc = (ntiles + want - 1) / want;
    a.nchunk = (ntiles + a.tpc - 1) / a.tpc;
    hipLaunchKernelGGL(k_wgrad3_f32, dim3(wg_grid(a)), dim3(256), 0, s, a);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_wgradT(WgradArgs<float>& a, int cap, hipStream_t s) {
    // 64 chunks: with 16 x 32 channel tiles 2 blocks per CU and more
    const int ntiles = (a.W + 7) / 8 * ((a.H + 7) / 8) * a.B, want = std::min(64, cap);
    a.nct = (a.cin_p + 31) / 32 * (a.cout_p / 16);
    a.tpc = (ntiles + want - 1) / want;
    a.nchunk = (ntiles + a.tpc - 1) / a.tpc;
    hipLaunchKernelGGL(k_wgradT_f32, dim3(wg_grid(a)), dim3(256), 0, s, a);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

}  // namespace hz
