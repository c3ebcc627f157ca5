// Launcher of the streamed-weights 3x3 convolution, instantiated once per precision.
#pragma once

#include "net_stream.h"

namespace hz {

template <class S, int NCB, int RPW, int WC, int WR>
static int launch_form(const Conv3sArgs<typename S::P>& g, hipStream_t s) {
    constexpr int TN = 16 * NCB * WC, TH = RPW * WR;
    const int64_t nblk = (int64_t)((g.W + 15) / 16) * ((g.H + TH - 1) / TH) * (g.cout_p / TN) * g.batch;
    if (nblk <= 0 || nblk > INT32_MAX) {
        set_error("conv3: grid too large");
        return HZ_ERR_ARG;
    }
    const dim3 grid((unsigned)nblk), block(64 * WC * WR);
#define HZ_CS(E)                                                                                                \
    hipLaunchKernelGGL((k_conv3s<S, NCB, RPW, WC, WR, E>), grid, block, 0, s, g.x0, g.c0, g.x1, g.c1, g.wf, g.bias, \
                       g.y, g.cout_p, g.ypool, g.H, g.W, g.relu, g.skip, g.ex)
    if (g.ex.head_w) {
        if constexpr (WC == 1) HZ_CS(CS_HEAD);
    } else if (g.ex.split || g.ex.mask0_ || g.ex.mask1_) {
        HZ_CS(CS_MASKED);
    } else if (g.ypool) {
        HZ_CS(CS_POOL);
    } else {
        HZ_CS(CS_PLAIN);
    }
#undef HZ_CS
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

template <class S>
static int launch_conv3s_any(int form, const Conv3sArgs<typename S::P>& g, hipStream_t s) {
    if (!conv3s_form_ok<typename S::P>(form, g.c0, g.c1, g.cout_p, g.ex.split, g.ex.head_w != nullptr) || !g.wf) {
        set_error("conv3: the streamed form does not take these channels");
        return HZ_ERR_ARG;
    }
    switch (form) {
#define HZ_CSF(ID, NCB, RPW, WC, WR) \
    case ID: return launch_form<S, NCB, RPW, WC, WR>(g, s);
        HZ_CONV3S_FORMS(HZ_CSF)
#undef HZ_CSF
    }
    set_error("conv3: unknown streamed form");
    return HZ_ERR_ARG;
}

template <class S, int NCB, int RPW, int WC, int WR>
static int launch_form_jobs(const TileJob* jobs, int njobs, const LayerIO* io, const void* wf, const float* bias, int c0,
                            int c1, int cout_p, bool pool, const typename S::P::T* head_w, const float* head_b, int col,
                            bool c128, hipStream_t s) {
#define HZ_CSJ(E)                                                                                                    \
    hipLaunchKernelGGL((k_conv3s_jobs<S, NCB, RPW, WC, WR, E>), dim3(njobs), dim3(64 * WC * WR), 0, s, jobs, io, wf, bias, \
                       c0, c1, cout_p, head_w, head_b, col, c128 ? 1 : 0)
    if (head_w) {
        if constexpr (WC == 1) HZ_CSJ(CS_HEAD);
    } else if (pool) {
        HZ_CSJ(CS_POOL);
    } else {
        HZ_CSJ(CS_PLAIN);
    }
#undef HZ_CSJ
    HZ_LAUNCH_CHECK();
    return HZ_OK;
}

template <class S>
static int launch_conv3s_jobs_any(int form, const TileJob* jobs, int njobs, const LayerIO* io, const void* wf,
                                  const float* bias, int c0, int c1, int cout_p, bool pool,
                                  const typename S::P::T* head_w, const float* head_b, int col, bool c128,
                                  hipStream_t s) {
    if (njobs <= 0) return HZ_OK;
    if (!conv3s_form_ok<typename S::P>(form, c0, c1, cout_p, 0, head_w != nullptr) || !wf || (head_w && pool)) {
        set_error("conv3 jobs: the streamed form does not take these channels");
        return HZ_ERR_ARG;
    }
    switch (form) {   // the forms conv3s_pick chooses from
#define HZ_CSF(ID, NCB, RPW, WC, WR)                                                                              \
    case ID:                                                                                                      \
        if constexpr (ID != 3 && ID != 6 && ID != 8 && ID != 13)                                                  \
            return launch_form_jobs<S, NCB, RPW, WC, WR>(jobs, njobs, io, wf, bias, c0, c1, cout_p, pool, head_w, \
                                                         head_b, col, c128, s);                                  \
        else break;
        HZ_CONV3S_FORMS(HZ_CSF)
#undef HZ_CSF
    }
    set_error("conv3 jobs: unknown streamed form");
    return HZ_ERR_ARG;
}

}  // namespace hz
