// Streamed-weights 3x3 convolution, BF16.
#include "net_stream_impl.h"

namespace hz {
template <>
int launch_conv3s<PolBF16>(int form, const Conv3sArgs<PolBF16>& g, hipStream_t s) {
    return launch_conv3s_any<StBF16>(form, g, s);
}
template <>
int launch_conv3s_jobs<PolBF16>(int form, const TileJob* jobs, int njobs, const LayerIO* io, const void* wf,
                            const float* bias, int c0, int c1, int cout_p, bool pool, const PolBF16::T* head_w,
                            const float* head_b, int col, bool c128, hipStream_t s) {
    return launch_conv3s_jobs_any<StBF16>(form, jobs, njobs, io, wf, bias, c0, c1, cout_p, pool, head_w, head_b, col, c128,
                                      s);
}
}  // namespace hz
