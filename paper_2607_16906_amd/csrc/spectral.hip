// Fourier-differentiation (pseudo-spectral) form of the Helmholtz operator with PML: the
// discretization of Section 2.1 / Table 1, derivatives over the whole grid taken as periodic.
//
// Per axis the spectral first derivative is the circulant matrix D[j][l] = d[(j - l) mod N] with
// d[0] = 0 and, for m != 0, d[m] = (pi / L) (-1)^m cot(pi m / N) (N even; the Nyquist mode's
// derivative vanishes at the nodes) or (pi / L) (-1)^m csc(pi m / N) (N odd), L = N h. With the
// stretching G = diag(1 / gamma), gamma = 1 + i sigma / omega at the nodes, the operator is
//     A u = u Mx^T + My u + k^2 u,   M = G D G D   (u as an [ny][nx] matrix),
// and A^H w = w conj(Mx) + My^H w + k^2 w. The library forms Mx and My once per problem
// (FP64 and FP32), so that one launch applies A: for the grids of this method (N up to a few
// thousand) the two per-axis contractions are dense complex GEMMs of 8 N FLOP per node each, run
// on the matrix cores, with no temporaries and no FFT passes.
#include "problem.h"

namespace hz {

// the circulant's first column: d[m], m = 0..n-1
__global__ void k_spec_table(double* d, int n, double h) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= n) return;
    if (m == 0) {
        d[0] = 0.0;
        return;
    }
    const double t = M_PI * m / n;
    const double f = (n % 2 == 0) ? cos(t) / sin(t) : 1.0 / sin(t);
    d[m] = (M_PI / (n * h)) * ((m & 1) ? -1.0 : 1.0) * f;
}

__device__ inline double2 inv_gamma(int i, int n, int npml, double omega, double sigma_max) {
    double sig = 0.0;
    if (npml > 0) {
        const double dep = fmax(0.0, fmax((double)(npml - i), (double)(i - (n - 1 - npml))));
        sig = sigma_max * (dep / npml) * (dep / npml);
    }
    // 1 / (1 + i s) = (1 - i s) / (1 + s^2), s = sigma / omega
    const double s = sig / omega;
    const double den = 1.0 + s * s;
    return double2{1.0 / den, -s / den};
}

// M[j][l] = g_j sum_k d[(j - k) mod n] g_k d[(k - l) mod n] (FP64), and its FP32 copy
__global__ void k_spec_mmat(double2* __restrict__ Md, float2* __restrict__ Mf, const double* __restrict__ d,
                            int n, int npml, double omega, double sigma_max) {
    const int l = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y;
    if (l >= n) return;
    double ar = 0.0, ai = 0.0;
    for (int k = 0; k < n; ++k) {
        const double dj = d[(j - k + n) % n];
        const double dl = d[(k - l + n) % n];
        const double2 gk = inv_gamma(k, n, npml, omega, sigma_max);
        const double c = dj * dl;
        ar += c * gk.x;
        ai += c * gk.y;
    }
    const double2 gj = inv_gamma(j, n, npml, omega, sigma_max);
    const double2 m{gj.x * ar - gj.y * ai, gj.x * ai + gj.y * ar};
    Md[(int64_t)j * n + l] = m;
    Mf[(int64_t)j * n + l] = float2{(float)m.x, (float)m.y};
}

// Matrix-core form. The two per-axis contractions are complex GEMMs, each taken as four real
// 16 x 16 x 4 MFMA products per k-step (re += a.re b.re - a.im b.im, im += a.re b.im + a.im b.re). Three products
// (sums and differences of the parts, 10 % to 20 % faster at 1088^2) would do, but their sums have the size of
// the larger part and cancel: with a part of 1e-2 of the other its error is 1e2 times as large.
// A block of 8 wavefronts owns a (16 NB) x (16 NB) output tile; wavefronts 0-3 form the x part sum_k
// u[y][k] Mx'[x][k], wavefronts 4-7 the y part sum_k My'[y][k] u[k][x], each over every fourth chunk
// of SPK k values. Operands go from memory straight into registers, the next chunk's while the matrix
// cores work: lane group g holds k values 4 g .. 4 g + 3 of a chunk and step s contracts the s-th of
// each group (the order of the contraction is free as long as both operands agree), so a lane reads
// 4 consecutive complex values of a row. The 8 partial tiles meet in LDS and are added in wavefront
// order; the epilogue adds k^2 u, and for RESID forms r = b - A u with the tile's ||r||^2 in
// part[tile]. Mx' = Mx and My' = My, or for ADJ Mx'[x][k] = conj(Mx[k][x]) and My'[y][k] =
// conj(My[k][y]). FP32 takes v_mfma_f32_16x16x4_f32, FP64 v_mfma_f64_16x16x4_f64.
//
// 32 x 32 tiles are bound by the matrix cores (64 instructions per 4 operands of 16 k values) and the
// rounds of tiles a CU takes one at a time; at small grids the chain of a block's chunks takes the time,
// which 16 x 16 tiles with a quarter of the chunks per wavefront shorten. Measured against 32 x 32 tiles
// staged in LDS with one chain per part: 296^2 20.2 -> 10.3 us FP32 (adjoint 23.2 -> 10.7), 30 -> 19 us FP64;
// 1088^2 234 -> 216 us FP32 (95 of 157 TFLOP/s; adjoint 274 -> 226), 375 -> 388 us FP64 (adjoint 423 -> 388). The
// error against 64 bits falls, too (FP32, 1088^2: 7.1e-7 -> 3.6e-7), from the shorter sums.
constexpr int SPK = 16;     // k values per chunk
constexpr int SPW = 512;    // threads per block

template <typename T>
struct SpecMma;
template <>
struct SpecMma<float> {
    typedef __attribute__((ext_vector_type(4))) float V;
    __device__ static V mma(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    __device__ static int row_of(int lg, int r) { return 4 * lg + r; }
};
template <>
struct SpecMma<double> {
    typedef __attribute__((ext_vector_type(4))) double V;
    __device__ static V mma(double a, double b, V c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    __device__ static int row_of(int lg, int r) { return lg + 4 * r; }
};

// 4 consecutive complex values of a row (FP32: 8-byte aligned, an odd row length leaves no more)
template <typename C>
__device__ __forceinline__ void load_row4(const C* p, C (&v)[4]) {
    if constexpr (sizeof(C) == 8) {
        typedef float f4_t __attribute__((ext_vector_type(4), aligned(8)));
        const f4_t a = *(const f4_t*)p, b = *(const f4_t*)(p + 2);
        v[0] = C{a.x, a.y};
        v[1] = C{a.z, a.w};
        v[2] = C{b.x, b.y};
        v[3] = C{b.z, b.w};
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = p[i];
    }
}

template <typename C, bool ADJ, bool RESID, int NB>
__global__ __launch_bounds__(SPW) void k_spectral(const C* __restrict__ u, C* __restrict__ y, const C* __restrict__ b,
                                                  const C* __restrict__ Mx, const C* __restrict__ My,
                                                  const decltype(C{}.x)* __restrict__ k2, int nx, int ny,
                                                  double* __restrict__ part, const int* __restrict__ skip) {
    using T = decltype(C{}.x);
    using M = SpecMma<T>;
    using V = typename M::V;
    if (skip && *skip) return;
    __shared__ T red[8][2][NB][256];      // one row of 16 x 16 blocks at a time: [wavefront][re/im][block][entry]
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // x / y part, every fourth chunk from kq on (shifted between the parts, so that the two wavefronts
    // of a SIMD do not both have the longer share)
    const int prt = wv >> 2, kq = (wv + 2 * prt) & 3;
    const int lr = lane & 15, lg = lane >> 4;
    const int x0 = blockIdx.x * 16 * NB, y0 = blockIdx.y * 16 * NB;
    const int nk = prt ? ny : nx;
    // rows and columns past the grid repeat the last one; their entries are not written
    int gy[NB], gx[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) gy[i] = min(y0 + 16 * i + lr, ny - 1);
#pragma unroll
    for (int i = 0; i < NB; ++i) gx[i] = min(x0 + 16 * i + lr, nx - 1);
    // operands of the chunk whose k values of this lane start at k: a[i] rows y0 + 16 i.., b[i] columns
    auto gload = [&](int k, bool whole, C (&a)[NB][4], C (&bb)[NB][4]) {
        if (whole) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (prt == 0) load_row4(u + (int64_t)gy[i] * nx + k, a[i]);
                else if (!ADJ) load_row4(My + (int64_t)gy[i] * ny + k, a[i]);
                else {
#pragma unroll
                    for (int s = 0; s < 4; ++s) a[i][s] = My[(int64_t)(k + s) * ny + gy[i]];
                }
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (prt == 0 && !ADJ) load_row4(Mx + (int64_t)gx[i] * nx + k, bb[i]);
                else {
                    const C* src = prt == 0 ? Mx : u;
#pragma unroll
                    for (int s = 0; s < 4; ++s) bb[i][s] = src[(int64_t)(k + s) * nx + gx[i]];
                }
            }
            return;
        }
        // the last chunk of a ragged length: zeros past its end
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int kl = k + s;
            const bool in = kl < nk;
            const int kk = in ? kl : 0;
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const C v = prt == 0 ? u[(int64_t)gy[i] * nx + kk]
                                     : (ADJ ? My[(int64_t)kk * ny + gy[i]] : My[(int64_t)gy[i] * ny + kk]);
                a[i][s] = in ? v : C{0, 0};
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const C v = prt == 0 ? (ADJ ? Mx[(int64_t)kk * nx + gx[i]] : Mx[(int64_t)gx[i] * nx + kk])
                                     : u[(int64_t)kk * nx + gx[i]];
                bb[i][s] = in ? v : C{0, 0};
            }
        }
    };
    V re[NB][NB], im[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) re[i][j][r] = im[i][j][r] = T(0);
    const int nch = (nk + SPK - 1) / SPK;
    // two operand sets in turn: one is loaded while the matrix cores work on the other
    C a0[NB][4], b0[NB][4], a1[NB][4], b1[NB][4];
    auto at = [&](int ch, C (&a)[NB][4], C (&bb)[NB][4]) {
        if (ch < nch) gload(ch * SPK + 4 * lg, (ch + 1) * SPK <= nk, a, bb);
    };
    // (the conjugated matrix of ADJ: My' is the first operand of the y part, Mx' the second of the x part)
    auto compute = [&](C (&a)[NB][4], C (&bb)[NB][4]) {
        if (ADJ) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    a[i][s].y = prt == 1 ? -a[i][s].y : a[i][s].y;
                    bb[i][s].y = prt == 0 ? -bb[i][s].y : bb[i][s].y;
                }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    re[i][j] = M::mma(a[i][s].x, bb[j][s].x, re[i][j]);
                    im[i][j] = M::mma(a[i][s].x, bb[j][s].y, im[i][j]);
                }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    re[i][j] = M::mma(-a[i][s].y, bb[j][s].y, re[i][j]);
                    im[i][j] = M::mma(a[i][s].y, bb[j][s].x, im[i][j]);
                }
        }
    };
    at(kq, a0, b0);
    for (int ch = kq; ch < nch; ch += 8) {
        at(ch + 4, a1, b1);
        compute(a0, b0);
        if (ch + 4 < nch) {
            at(ch + 8, a0, b0);
            compute(a1, b1);
        }
    }
    // add the 8 partial tiles, one row of 16 x 16 blocks at a time: thread t finishes entry t % 256 (row
    // t / 16 % 16, column t % 16) of block t / 256
    double nrm = 0.0;
    const int j = threadIdx.x >> 8, e = threadIdx.x & 255;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        if (i) __syncthreads();
#pragma unroll
        for (int jj = 0; jj < NB; ++jj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int pos = M::row_of(lg, r) * 16 + lr;
                red[wv][0][jj][pos] = re[i][jj][r];
                red[wv][1][jj][pos] = im[i][jj][r];
            }
        __syncthreads();
        const int oy = y0 + 16 * i + (e >> 4), ox = x0 + 16 * j + (e & 15);
        if (j < NB && oy < ny && ox < nx) {
            T vr = red[0][0][j][e], vi = red[0][1][j][e];
#pragma unroll
            for (int w = 1; w < 8; ++w) {
                vr += red[w][0][j][e];
                vi += red[w][1][j][e];
            }
            const int64_t idx = (int64_t)oy * nx + ox;
            const C uq = u[idx];
            const T kq2 = k2[idx];
            vr += kq2 * uq.x;
            vi += kq2 * uq.y;
            if (RESID) {
                vr = b[idx].x - vr;
                vi = b[idx].y - vi;
                nrm += (double)vr * vr + (double)vi * vi;
            }
            y[idx] = C{vr, vi};
        }
    }
    if (RESID) {
        __shared__ double rn[SPW / 64];
        const double t = wave_sum(nrm);
        if (lane == 0) rn[wv] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            double acc = 0.0;
#pragma unroll
            for (int w = 0; w < SPW / 64; ++w) acc += rn[w];
            part[blockIdx.y * gridDim.x + blockIdx.x] = acc;
        }
    }
}

// Edge of a grid's tiles in 16 x 16 blocks: 2 or 1. A CU runs one block at a time, so a launch takes
// its tiles in rounds of 256; a small tile takes about 6/5 of a quarter of a large one's time (fewer
// matrix instructions per load): 544^2, 289 large tiles in two rounds 49 us, 1156 small ones in five
// 37 us; 488^2, 256 large ones in one round 25 us, 961 small ones 26 us (FP32; FP64 86, 67, 43 and 51 us).
static int spectral_nb(const hz_problem* p) {
    auto rounds = [&](int te) {
        const int64_t t = (int64_t)((p->nxt + te - 1) / te) * ((p->nyt + te - 1) / te);
        return (t + 255) / 256;
    };
    return rounds(32) * 4 * 5 <= rounds(16) * 6 ? 2 : 1;
}

static dim3 spectral_grid(const hz_problem* p) {
    const int te = 16 * spectral_nb(p);
    return dim3((p->nxt + te - 1) / te, (p->nyt + te - 1) / te);
}

int spectral_blocks(const hz_problem* p) {
    const dim3 g = spectral_grid(p);
    return (int)(g.x * g.y);
}

int spectral_setup(hz_problem* p, hipStream_t s) {
    const hz_grid& g = p->g;
    hipLaunchKernelGGL(k_spec_table, dim3((p->nxt + 127) / 128), dim3(128), 0, s, p->dtx, p->nxt, g.h);
    hipLaunchKernelGGL(k_spec_table, dim3((p->nyt + 127) / 128), dim3(128), 0, s, p->dty, p->nyt, g.h);
    hipLaunchKernelGGL(k_spec_mmat, dim3((p->nxt + 127) / 128, p->nxt), dim3(128), 0, s, p->Mx_d, p->Mx_f, p->dtx,
                       p->nxt, g.npml, g.omega, g.sigma_max);
    hipLaunchKernelGGL(k_spec_mmat, dim3((p->nyt + 127) / 128, p->nyt), dim3(128), 0, s, p->My_d, p->My_f, p->dty,
                       p->nyt, g.npml, g.omega, g.sigma_max);
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

template <typename C, bool ADJ, bool RESID>
static int launch_tile(const hz_problem* p, const C* x, C* y, const C* b, const C* Mx, const C* My,
                       const decltype(C{}.x)* k2, double* part, const int* skip, hipStream_t s) {
    const dim3 g = spectral_grid(p);
#define HZ_SP(NB)                                                                                                  \
    hipLaunchKernelGGL((k_spectral<C, ADJ, RESID, NB>), g, dim3(SPW), 0, s, x, y, b, Mx, My, k2, p->nxt, p->nyt, \
                       part, skip)
    if (spectral_nb(p) == 2) HZ_SP(2);
    else HZ_SP(1);
#undef HZ_SP
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

int launch_spectral(const hz_problem* p, bool fp64, bool adjoint, const void* x, void* y, hipStream_t s,
                    const int* skip) {
    if (fp64) {
        const double2 *xd = (const double2*)x, *Mx = (const double2*)p->Mx_d, *My = (const double2*)p->My_d;
        return adjoint ? launch_tile<double2, true, false>(p, xd, (double2*)y, nullptr, Mx, My, p->k2d, nullptr, skip, s)
                       : launch_tile<double2, false, false>(p, xd, (double2*)y, nullptr, Mx, My, p->k2d, nullptr, skip, s);
    }
    const float2 *xf = (const float2*)x, *Mx = (const float2*)p->Mx_f, *My = (const float2*)p->My_f;
    return adjoint ? launch_tile<float2, true, false>(p, xf, (float2*)y, nullptr, Mx, My, p->k2f, nullptr, skip, s)
                   : launch_tile<float2, false, false>(p, xf, (float2*)y, nullptr, Mx, My, p->k2f, nullptr, skip, s);
}

int launch_spectral_resid32(const hz_problem* p, const float2* b, const float2* x, float2* r, double* part,
                            const int* skip, hipStream_t s) {
    return launch_tile<float2, false, true>(p, x, r, b, (const float2*)p->Mx_f, (const float2*)p->My_f, p->k2f, part,
                                            skip, s);
}

int launch_spectral_resid64(const hz_problem* p, const double2* b, const double2* x, double2* r, double* part,
                            const int* skip, hipStream_t s) {
    return launch_tile<double2, false, true>(p, x, r, b, (const double2*)p->Mx_d, (const double2*)p->My_d, p->k2d, part,
                                             skip, s);
}

}  // namespace hz
