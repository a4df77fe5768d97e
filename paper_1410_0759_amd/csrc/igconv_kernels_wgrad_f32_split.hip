// fp32 backward-filter kernels on the bfloat16 matrix pipes, every operand split into three parts
// (igconv_kernel_wgrad_f32s.hpp).
#include "igconv_kernel_wgrad_f32s.hpp"

namespace igc {

template <class Cfg>
static int launch_wgrad_f32s(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_wgrad_f32s_kernel<Cfg>, "igconv_wgrad_f32s_kernel", p, grid, Cfg::THREADS, stream);
}

//    name, BM, BN, WM, WN
#define IGC_WGRAD_F32S_LIST(X) \
    X("f32 64x128x32 wgrad split tap", 64, 128, 2, 2) \
    X("f32 96x128x32 wgrad split tap", 96, 128, 1, 4) \
    X("f32 128x64x32 wgrad split tap", 128, 64, 2, 2) \
    X("f32 128x128x32 wgrad split tap", 128, 128, 2, 2)

#define IGC_WGRAD_F32S_INSTANTIATE(NAME, BM, BN, WM, WN) \
    template __global__ void igconv_wgrad_f32s_kernel<WgradSplitConfig<BM, BN, WM, WN>>(const ConvKernelParams);
IGC_WGRAD_F32S_LIST(IGC_WGRAD_F32S_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
// (variant 4: operands split)
#define IGC_WGRAD_F32S_ROW(NAME, BM, BN, WM, WN)                                       \
    {NAME, false, BM, BN, 32, false, false, GATHER_WGRAD_TAP, WgradSplitConfig<BM, BN, WM, WN>::THREADS, \
     WgradSplitConfig<BM, BN, WM, WN>::LDS_BYTES, &launch_wgrad_f32s<WgradSplitConfig<BM, BN, WM, WN>>, 4},
static const KernelInfo kRows[] = {IGC_WGRAD_F32S_LIST(IGC_WGRAD_F32S_ROW)};
const KernelGroup kGroupWgradF32Split = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
