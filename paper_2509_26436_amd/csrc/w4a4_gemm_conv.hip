// W4A4 GEMM instantiations: the 3 x 3 convolution as an implicit GEMM, in the
// per-group and in the static (LDM) setting.
#include "w4a4_gemm_kernel.h"

namespace quartz {
namespace {

// The per-group convolution takes the tile that the linear layer takes on the
// im2col matrix (with or without its split, as a workspace is there): both
// then add the groups in the same order, so their outputs are equal bit for
// bit.  (4096 x 5760 -> 640: 37 us against 44 on w4a4_gemm; 9216 x 5760 ->
// 1280: 88 against 104; where the linear layer stays with w4a4_linear, w4a4_gemm
// wins here too: 16384 x 2880 -> 320 34 against 38.)  The static one's sums
// are exact integers in any order (26 us against 41; 53 against 86; 27 against
// 31).
WideShape conv_shape(const GemmLaunch& a, WideMode mode)
{
    return wide_shape(a.M, a.N, a.K, mode,
                      linear_schedule(a.M, a.N, a.K, linear_resident_blocks(), a.counters != nullptr), true);
}

}  // namespace

hipError_t launch_gemm_conv(const GemmLaunch& a, hipStream_t stream)
{
    if (const WideShape w = conv_shape(a, WideMode::kPlain); w.tr > 0)
        return launch_wide_conv(a, w, stream);
    return launch_mode<false, false, true>(a, stream);
}

hipError_t launch_gemm_conv_static(const GemmLaunch& a, hipStream_t stream)
{
    if (const WideShape w = conv_shape(a, WideMode::kStatic); w.tr > 0)
        return launch_wide_conv_static(a, w, stream);
    return launch_mode<false, true, true>(a, stream);
}

}  // namespace quartz
