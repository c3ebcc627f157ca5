// Weight gradients on the matrix cores (train_wgrad.hip).
#pragma once
#include "net_kernels.h"

namespace hz {

template <class T>
struct WgradArgs {
    const T* G;            // 3x3: [B][H][W][cout_p]; transposed: [B][2H][2W][cout_p]
    const T *x0, *x1;      // input [B][H][W]: channels [0, c0) in x0, [c0, cin_p) in x1
    int c0, cin_p, cout_p;
    int B, H, W;
    float *part, *partb;   // [nchunk][taps][cout_p][cin_p], [nchunk][cout_p]
    int tpc, nchunk, nct;  // tiles per chunk, chunks, channel tiles (set by the launch)
};

// 3x3 and transposed 2x2 weight gradients into at most cap chunks of partials; sets a.nchunk.
int launch_wgrad3(WgradArgs<bf16_t>& a, int cap, hipStream_t s);
int launch_wgrad3(WgradArgs<float>& a, int cap, hipStream_t s);
int launch_wgradT(WgradArgs<bf16_t>& a, int cap, hipStream_t s);
int launch_wgradT(WgradArgs<float>& a, int cap, hipStream_t s);

}  // namespace hz
