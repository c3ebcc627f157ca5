// Level 0 of the U-Net in two launches (BF16, 32 base channels, inference): its encoder pair and its
// decoder with the output head. Every intermediate tensor of the level stays in LDS.
//
//   encoder: X (8 channels) -> 3x3 + ReLU -> 3x3 + ReLU -> E (and its 2x2 average pool)
//   decoder: D (64 channels, half the size) -> 2x2 transposed -> U; [E, U] -> 3x3 + ReLU -> 3x3 + ReLU -> head z
//
// Level 0 has the most pixels and the fewest channels: as separate layers it is bound by the bytes
// its tensors move (6 of 32 channels each way at full size) and, on small grids, by the latency of
// its 5 launches. A block of 4 wavefronts owns a 14 x 14 tile of outputs: the inner layer covers 16 x
// 16 pixels (one 16-pixel matrix column block per row, 4 rows per wavefront) and its input 18 x 18,
// so both layers run the same regular tile; 30 % of the matrix work is on the overlap, which costs
// less than the tensors. Every sum has the operands and order of the separate layers and every
// intermediate is rounded as it would be stored (the same result bits).
//
// Measured, separate -> fused: 1088^2 encoder 84 -> 44 us, decoder 171 -> 100 us (700 -> 241 MB of memory traffic,
// 237 without repeats); 296^2 17 -> 8 us and 21 -> 13 us. Bound by the phases of a block, which wait for each
// other at barriers: the matrix cores are busy for 33 and 39 % of the cycles, the LDS for 29 and 39 %.
#include "net_stream.h"

namespace hz {

constexpr int L0_TILE = LEVEL0_TILE;
constexpr int L0_NT = 256;
constexpr int L0_PATCH = 18 * 18 * CS_PB;   // bytes of an 18 x 18 patch of one 32-channel chunk

// One 9-tap chunk over a patch in LDS: the wavefront's 4 rows of 2 x 16 channels (as conv3s_tile with
// RPW = 4, NCB = 2). a holds 3 taps of operands; tap + 3 is loaded from wk, past the chunk from wn.
__device__ __forceinline__ void l0_chunk(f32x4_t (&acc)[4][2], uint4 (&a)[3][2], const unsigned char* pb,
                                         const unsigned char* wk, const unsigned char* wn) {
    uint4 b[6][3];
    auto bload = [&](int row, int dx) { return *(const uint4*)(pb + (row * 18 + dx) * CS_PB); };
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r][0] = bload(r, 0);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int dy = tap / 3, dx = tap % 3;
        if (tap + 1 < 9) {
            const int ny = (tap + 1) / 3, nx = (tap + 1) % 3;
            if (ny == 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) b[r][nx] = bload(r, nx);
            } else {
                b[4 + ny - 1][nx] = bload(4 + ny - 1, nx);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[r][cb] = StBF16::mma(a[tap % 3][cb], b[r + dy][dx], acc[r][cb], 0);
        const int nt = tap + 3;
        const unsigned char* w = nt < 9 ? wk : wn;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) a[tap % 3][cb] = *(const uint4*)(w + (cb * 9 + nt % 9) * 1024);
        __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ __forceinline__ void l0_zero(f32x4_t (&acc)[4][2]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) acc[r][cb] = f32x4_t{0, 0, 0, 0};
}

// The inner layer's rows into the patch of the outer one: bias, ReLU, rounding; zero outside the image.
// Row 4 wv + r, column lr of the 16 x 16 tile at (y0, x0) is patch pixel (4 wv + r, lr).
__device__ __forceinline__ void l0_store_inner(const f32x4_t (&acc)[4][2], const float (&bv)[2][4], unsigned char* patch,
                                               int y0, int x0, int H, int W, int wv, int lr, int lg) {
    const int gx = x0 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int gy = y0 + 4 * wv + r;
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            float t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float s = acc[r][cb][q] + bv[cb][q];
                t[q] = s > 0.0f ? s : 0.0f;
            }
            *(uint2*)(patch + ((4 * wv + r) * 18 + lr) * CS_PB + cb * 32 + 8 * lg) =
                in ? uint2{f2bf_pair(t[0], t[1]), f2bf_pair(t[2], t[3])} : uint2{0, 0};
        }
    }
}

__device__ __forceinline__ void l0_bias(const float* bias, int lg, float (&bv)[2][4]) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) bv[cb][q] = bias[cb * 16 + 4 * lg + q];
}

__device__ __forceinline__ void l0_encoder(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wa,
                                           const float* __restrict__ ba, const void* __restrict__ wfb,
                                           const float* __restrict__ bb, bf16_t* __restrict__ y,
                                           bf16_t* __restrict__ ypool, int H, int W, int ty0, int tx0, int skipped) {
    __shared__ __attribute__((aligned(16))) unsigned char xp[18 * 18 * 16];
    __shared__ __attribute__((aligned(16))) unsigned char tp[L0_PATCH];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    // input patch at (ty0 - 2, tx0 - 2): one 16-byte vector per pixel
    uint4 rx[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int px = min((int)threadIdx.x + i * L0_NT, 18 * 18 - 1);
        const int gy = ty0 - 2 + px / 18, gx = tx0 - 2 + px % 18;
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
        const uint4 v = *(const uint4*)(x + (in ? (int64_t)gy * W + gx : 0) * 8);
        rx[i] = in ? v : uint4{0, 0, 0, 0};
    }
    // first layer's operands: step s, lane group lg: tap 4 s + lg (zero past the ninth)
    uint4 a8[3][2];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int tap = 4 * s + lg;
            const uint4 v = *(const uint4*)(wa + (min(tap, 8) * 32 + cb * 16 + lr) * 8);
            a8[s][cb] = tap < 9 ? v : uint4{0, 0, 0, 0};
        }
    const unsigned char* wk = (const unsigned char*)wfb + lane * 16;
    uint4 a[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) a[t][cb] = *(const uint4*)(wk + (cb * 9 + t) * 1024);
    float bva[2][4], bvb[2][4];
    l0_bias(ba, lg, bva);
    l0_bias(bb, lg, bvb);
    asm volatile("" ::: "memory");   // keep the loads above the test
    if (skipped) return;             // uniform over the block
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int px = (int)threadIdx.x + i * L0_NT;
        if (px < 18 * 18) *(uint4*)(xp + px * 16) = rx[i];
    }
    __syncthreads();
    f32x4_t acc[4][2];
    l0_zero(acc);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int tap = min(4 * s + lg, 8);   // (the operand of a tap past the ninth is zeroed)
        const int dy = tap / 3, dx = tap - 3 * dy;
        const bool live = 4 * s + lg < 9;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            uint4 b = *(const uint4*)(xp + ((4 * wv + r + dy) * 18 + lr + dx) * 16);
            if (!live) b = uint4{0, 0, 0, 0};
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[r][cb] = StBF16::mma(a8[s][cb], b, acc[r][cb], 0);
        }
    }
    l0_store_inner(acc, bva, tp, ty0 - 1, tx0 - 1, H, W, wv, lr, lg);
    __syncthreads();
    // (patch rows and columns 16 and 17 hold nothing: only outputs past the 14 x 14 tile read them)
    l0_zero(acc);
    l0_chunk(acc, a, tp + ((4 * wv) * 18 + lr) * CS_PB + lg * 16, wk, wk);
    const int gx = tx0 + lr;
    const bool colin = lr < L0_TILE && gx < W;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
        float v[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float t = acc[r][cb][q] + bvb[cb][q];
                v[r][q] = t > 0.0f ? t : 0.0f;
            }
            const int gy = ty0 + 4 * wv + r;
            if (colin && 4 * wv + r < L0_TILE && gy < H)
                PolBF16::store4(y + ((int64_t)gy * W + gx) * 32 + cb * 16 + 4 * lg, v[r]);
        }
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
            float p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float s = v[r][q] + v[r + 1][q];
                s += __shfl_xor(s, 1, 64);
                p[q] = 0.25f * s;
            }
            const int gy = ty0 + 4 * wv + r;
            if ((lr & 1) == 0 && colin && 4 * wv + r < L0_TILE && gy < H)
                PolBF16::store4(ypool + ((int64_t)(gy / 2) * (W / 2) + gx / 2) * 32 + cb * 16 + 4 * lg, p);
        }
    }
}

__device__ __forceinline__ void l0_decoder(const bf16_t* __restrict__ e, const bf16_t* __restrict__ d,
                                           const Level0Dec& w, int H, int W, int ty0, int tx0, void* z, int c128,
                                           int nxt, int nyt, double fixed_s, const double* __restrict__ sc,
                                           int skipped) {
    constexpr int DPX = 81, DPS = 144;   // coarse patch: 9 x 9 pixels of 64 channels (+ 16 B against bank conflicts)
    static_assert(96 * DPS <= L0_PATCH, "the coarse patch shares the E patch's LDS");
    __shared__ __attribute__((aligned(16))) unsigned char pa[L0_PATCH];   // coarse patch, then E, then the inner layer
    __shared__ __attribute__((aligned(16))) unsigned char pu[L0_PATCH];   // U
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int Hd = H / 2, Wd = W / 2, dy0 = ty0 / 2 - 1, dx0 = tx0 / 2 - 1;
    // coarse patch (every channel): 8 vectors per pixel
    uint4 rd[3];
    uint32_t okd = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int u = min((int)threadIdx.x + i * L0_NT, DPX * 8 - 1);
        const int px = u >> 3, gy = dy0 + px / 9, gx = dx0 + px % 9;
        const bool in = gy >= 0 && gy < Hd && gx >= 0 && gx < Wd;
        okd |= (in ? 1u : 0u) << i;
        rd[i] = *(const uint4*)(d + (in ? (int64_t)gy * Wd + gx : 0) * 64 + (u & 7) * 8);
    }
    // transposed layer's operands of this wavefront's parity: 2 channel blocks x 2 K operands
    const int py = wv >> 1, px2 = wv & 1;
    const unsigned char* wt = (const unsigned char*)w.wfu + lane * 16;
    uint4 at[2][2];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int k = 0; k < 2; ++k) at[cb][k] = *(const uint4*)(wt + ((((py * 2 + cb) * 2 + px2) * 2) + k) * 1024);
    float bvu[2][4];
    l0_bias(w.bu, lg, bvu);
    // E patch at (ty0 - 2, tx0 - 2): 4 vectors per pixel
    uint4 re[6];
    uint32_t oke = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int u = min((int)threadIdx.x + i * L0_NT, 18 * 18 * 4 - 1);
        const int px = u >> 2, gy = ty0 - 2 + px / 18, gx = tx0 - 2 + px % 18;
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
        oke |= (in ? 1u : 0u) << i;
        re[i] = *(const uint4*)(e + (in ? (int64_t)gy * W + gx : 0) * 32 + (u & 3) * 8);
    }
    // inner layer: chunk 0 (E) and 1 (U), then the outer layer's chunk
    const unsigned char* wa0 = (const unsigned char*)w.wfa + lane * 16;
    const unsigned char* wa1 = wa0 + 2 * 9 * 1024;
    const unsigned char* wb0 = (const unsigned char*)w.wfb + lane * 16;
    uint4 a[3][2];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) a[t][cb] = *(const uint4*)(wa0 + (cb * 9 + t) * 1024);
    asm volatile("" ::: "memory");   // keep the loads above the test
    if (skipped) return;             // uniform over the block
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int u = (int)threadIdx.x + i * L0_NT;
        if (u < DPX * 8)
            *(uint4*)(pa + (u >> 3) * DPS + (u & 7) * 16) = ((okd >> i) & 1u) ? rd[i] : uint4{0, 0, 0, 0};
    }
    __syncthreads();
    // U: this parity's pixels of the 18 x 18 patch, zero outside the image
#pragma unroll
    for (int g = 0; g < 6; ++g) {
        const int n = g * 16 + lr;   // coarse pixel (columns past the 81st are computed and dropped)
        f32x4_t u[2] = {f32x4_t{0, 0, 0, 0}, f32x4_t{0, 0, 0, 0}};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint4 b = *(const uint4*)(pa + n * DPS + k * 64 + lg * 16);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) u[cb] = StBF16::mma(at[cb][k], b, u[cb], 0);
        }
        const int fy = 2 * (n / 9) + py, fx = 2 * (n % 9) + px2;
        const int gy = ty0 - 2 + fy, gx = tx0 - 2 + fx;
        const bool in = gy >= 0 && gy < H && gx >= 0 && gx < W;
        if (n < DPX) {
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                float t[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) t[q] = u[cb][q] + bvu[cb][q];
                *(uint2*)(pu + (fy * 18 + fx) * CS_PB + cb * 32 + 8 * lg) =
                    in ? uint2{f2bf_pair(t[0], t[1]), f2bf_pair(t[2], t[3])} : uint2{0, 0};
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int u = (int)threadIdx.x + i * L0_NT;
        if (u < 18 * 18 * 4)
            *(uint4*)(pa + (u >> 2) * CS_PB + (u & 3) * 16) = ((oke >> i) & 1u) ? re[i] : uint4{0, 0, 0, 0};
    }
    float bva[2][4];
    l0_bias(w.ba, lg, bva);
    __syncthreads();
    f32x4_t acc[4][2];
    l0_zero(acc);
    const int off = ((4 * wv) * 18 + lr) * CS_PB + lg * 16;
    l0_chunk(acc, a, pa + off, wa0, wa1);
    l0_chunk(acc, a, pu + off, wa1, wb0);
    __syncthreads();   // every wavefront has read the E patch
    l0_store_inner(acc, bva, pa, ty0 - 1, tx0 - 1, H, W, wv, lr, lg);
    __syncthreads();
    l0_zero(acc);
    l0_chunk(acc, a, pa + off, wb0, wb0);
    // output head over the 32 channels of a pixel, as conv3_tile's
    float o0[4], o1[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) o0[r] = o1[r] = 0.0f;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int co = cb * 16 + 4 * lg + q;
            const float w0 = bf2f(w.head_w[co]), w1 = bf2f(w.head_w[32 + co]), bc = w.bb[co];
            float t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] = acc[r][cb][q] + bc;
                t[r] = t[r] > 0.0f ? t[r] : 0.0f;
            }
#pragma unroll
            for (int r = 0; r < 4; r += 2) {   // rounded as stored
                const uint32_t u = f2bf_pair(t[r], t[r + 1]);
                const float lo = __builtin_bit_cast(float, u << 16), hi = __builtin_bit_cast(float, u & 0xffff0000u);
                o0[r] += lo * w0;
                o1[r] += lo * w1;
                o0[r + 1] += hi * w0;
                o1[r + 1] += hi * w1;
            }
        }
    const float hb0 = w.head_b[0], hb1 = w.head_b[1];
    const double sfac = fixed_s > 0 ? fixed_s : sc[0];
    const int gx = tx0 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float a0 = o0[r], a1 = o1[r];
        a0 += __shfl_xor(a0, 16, 64);
        a1 += __shfl_xor(a1, 16, 64);
        a0 += __shfl_xor(a0, 32, 64);
        a1 += __shfl_xor(a1, 32, 64);
        const int gy = ty0 + 4 * wv + r;
        if (lg == 0 && lr < L0_TILE && 4 * wv + r < L0_TILE && gy < nyt && gx < nxt) {
            const double2 zv{sfac * (double)(hb0 + a0), sfac * (double)(hb1 + a1)};
            const int64_t zi = (int64_t)gy * nxt + gx;
            if (c128) ((double2*)z)[zi] = zv;
            else ((float2*)z)[zi] = from_d2<float2>(zv);
        }
    }
}

__global__ __launch_bounds__(L0_NT, 2) void k_level0_enc(const bf16_t* __restrict__ x, Level0Enc w, bf16_t* __restrict__ y,
                                                         bf16_t* __restrict__ ypool, int H, int W,
                                                         const int* __restrict__ skip) {
    const int skipped = skip ? *skip : 0;
    const int ntx = (W + L0_TILE - 1) / L0_TILE;
    const int v = xcd_linear(blockIdx.x, gridDim.x);
    l0_encoder(x, w.wa, w.ba, w.wfb, w.bb, y, ypool, H, W, v / ntx * L0_TILE, v % ntx * L0_TILE, skipped);
}

__global__ __launch_bounds__(L0_NT, 2) void k_level0_dec(const bf16_t* __restrict__ e, const bf16_t* __restrict__ d,
                                                         Level0Dec w, int H, int W, void* z, int c128, int nxt, int nyt,
                                                         double fixed_s, const double* __restrict__ sc,
                                                         const int* __restrict__ skip) {
    const int skipped = skip ? *skip : 0;
    const int ntx = (W + L0_TILE - 1) / L0_TILE;
    const int v = xcd_linear(blockIdx.x, gridDim.x);
    l0_decoder(e, d, w, H, W, v / ntx * L0_TILE, v % ntx * L0_TILE, z, c128, nxt, nyt, fixed_s, sc, skipped);
}

// Ragged batch: job = (system, -, tile row, tile column).
__global__ __launch_bounds__(L0_NT, 2) void k_level0_enc_jobs(const TileJob* __restrict__ jobs,
                                                              const LayerIO* __restrict__ io, Level0Enc w) {
    const TileJob jb = jobs[xcd_linear(blockIdx.x, gridDim.x)];
    const LayerIO t = io[jb.sys];
    if (t.stop && *t.stop) return;
    l0_encoder((const bf16_t*)t.x0, w.wa, w.ba, w.wfb, w.bb, (bf16_t*)t.y, (bf16_t*)t.ypool, t.H, t.W, jb.ty0, jb.tx0, 0);
}

__global__ __launch_bounds__(L0_NT, 2) void k_level0_dec_jobs(const TileJob* __restrict__ jobs,
                                                              const LayerIO* __restrict__ io, Level0Dec w, int col,
                                                              int c128) {
    const TileJob jb = jobs[xcd_linear(blockIdx.x, gridDim.x)];
    const LayerIO t = io[jb.sys];
    if (t.stop && *t.stop) return;
    void* z = c128 ? (void*)((double2*)t.z + (int64_t)col * t.zld) : (void*)((float2*)t.z + (int64_t)col * t.zld);
    l0_decoder((const bf16_t*)t.x0, (const bf16_t*)t.x1, w, t.H, t.W, jb.ty0, jb.tx0, z, c128, t.nxt, t.nyt, 0.0, t.sc, 0);
}

static int check_grid(int64_t nblk, int H, int W) {
    if (nblk > INT32_MAX || H < 2 || W < 2 || H % 2 || W % 2) {
        set_error("level 0: bad grid");
        return HZ_ERR_ARG;
    }
    return HZ_OK;
}

int launch_level0_enc(const bf16_t* x, const Level0Enc& w, bf16_t* y, bf16_t* ypool, int H, int W, const int* skip,
                      hipStream_t s) {
    const int64_t nblk = (int64_t)((W + L0_TILE - 1) / L0_TILE) * ((H + L0_TILE - 1) / L0_TILE);
    HZ_TRY(check_grid(nblk, H, W));
    hipLaunchKernelGGL(k_level0_enc, dim3((unsigned)nblk), dim3(L0_NT), 0, s, x, w, y, ypool, H, W, skip);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_level0_dec(const bf16_t* e, const bf16_t* d, const Level0Dec& w, int H, int W, const Conv3Out& head,
                      const int* skip, hipStream_t s) {
    const int64_t nblk = (int64_t)((W + L0_TILE - 1) / L0_TILE) * ((H + L0_TILE - 1) / L0_TILE);
    HZ_TRY(check_grid(nblk, H, W));
    hipLaunchKernelGGL(k_level0_dec, dim3((unsigned)nblk), dim3(L0_NT), 0, s, e, d, w, H, W, head.head_z, head.head_c128,
                       head.head_nxt, head.head_nyt, head.head_fixed_s, head.head_sc, skip);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_level0_enc_jobs(const TileJob* jobs, int njobs, const LayerIO* io, const Level0Enc& w, hipStream_t s) {
    if (njobs <= 0) return HZ_OK;
    hipLaunchKernelGGL(k_level0_enc_jobs, dim3(njobs), dim3(L0_NT), 0, s, jobs, io, w);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_level0_dec_jobs(const TileJob* jobs, int njobs, const LayerIO* io, const Level0Dec& w, int col, bool c128,
                           hipStream_t s) {
    if (njobs <= 0) return HZ_OK;
    hipLaunchKernelGGL(k_level0_dec_jobs, dim3(njobs), dim3(L0_NT), 0, s, jobs, io, w, col, c128 ? 1 : 0);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

}  // namespace hz
