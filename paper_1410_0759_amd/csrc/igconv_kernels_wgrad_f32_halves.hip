// fp32 backward-filter kernels on the 16-bit matrix pipes, every operand as two binary16 parts (igconv_kernel_wgrad_f32h.hpp).
#include "igconv_kernel_wgrad_f32h.hpp"

namespace igc {

template <class Cfg>
static int launch_wgrad_f32h(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_wgrad_f32h_kernel<Cfg>, "igconv_wgrad_f32h_kernel", p, grid, Cfg::THREADS, stream);
}

//    name, channel-fastest tensors
#define IGC_WGRAD_F32H_LIST(X) \
    X("f32 64x64x128 wgrad halves", false) \
    X("f32 64x64x128 wgrad halves, channels innermost", true)

#define IGC_WGRAD_F32H_INSTANTIATE(NAME, NHWC) \
    template __global__ void igconv_wgrad_f32h_kernel<WgradHalvesConfig<NHWC>>(const ConvKernelParams);
IGC_WGRAD_F32H_LIST(IGC_WGRAD_F32H_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
// (variant 9: operands as two binary16 parts, three taps of a filter row per tile)
#define IGC_WGRAD_F32H_ROW(NAME, NHWC)                                                                                  \
    {NAME, false, 64, 64, 128, NHWC, false, GATHER_WGRAD_TAP, 512, WgradHalvesConfig<NHWC>::LDS_BYTES, \
     &launch_wgrad_f32h<WgradHalvesConfig<NHWC>>, 9},
static const KernelInfo kRows[] = {IGC_WGRAD_F32H_LIST(IGC_WGRAD_F32H_ROW)};
const KernelGroup kGroupWgradF32Halves = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
