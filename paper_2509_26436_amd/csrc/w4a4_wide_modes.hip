// The wide linear kernel (w4a4_wide_kernel.h) in the LDM setting and the
// asymmetric mode, a translation unit of their own so they compile in parallel.
#include "w4a4_wide_kernel.h"

namespace quartz {

hipError_t launch_wide_static(const GemmLaunch& a, hipStream_t stream)
{
    return launch_wide_mode<true, false, false, false>(a, stream);
}

hipError_t launch_wide_asym(const GemmLaunch& a, hipStream_t stream)
{
    return launch_wide_mode<false, false, true, false>(a, stream);
}

}  // namespace quartz
