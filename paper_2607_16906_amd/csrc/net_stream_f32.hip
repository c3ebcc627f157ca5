// Streamed-weights 3x3 convolution, FP32.
#include "net_stream_impl.h"

namespace hz {
template <>
int launch_conv3s<PolF32>(int form, const Conv3sArgs<PolF32>& g, hipStream_t s) {
    return launch_conv3s_any<StF32>(form, g, s);
}
}  // namespace hz
