// The wide linear kernel (w4a4_wide_kernel.h) on a 3 x 3 convolution, both
// settings.
#include "w4a4_wide_kernel.h"

namespace quartz {

hipError_t launch_wide_conv(const GemmLaunch& a, hipStream_t stream)
{
    return launch_wide_mode<false, false, false, true>(a, stream);
}

hipError_t launch_wide_conv_static(const GemmLaunch& a, hipStream_t stream)
{
    return launch_wide_mode<true, false, false, true>(a, stream);
}

}  // namespace quartz
