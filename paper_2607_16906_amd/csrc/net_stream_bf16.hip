// Streamed-weights 3x3 convolution, BF16.
#include "net_stream_impl.h"

namespace hz {
template <>
int launch_conv3s<PolBF16>(int form, const Conv3sArgs<PolBF16>& g, hipStream_t s) {
    return launch_conv3s_any<StBF16>(form, g, s);
}
}  // namespace hz
