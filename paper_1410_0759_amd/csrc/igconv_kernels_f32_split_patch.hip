// fp32 nine-tap kernels on the bfloat16 matrix pipes with a staged image patch (igconv_kernel_f32p.hpp).
#include "igconv_kernel_f32p.hpp"

namespace igc {

template <class Cfg>
static int launch_f32p(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_f32p_kernel<Cfg>, "igconv_f32p_kernel", p, grid, Cfg::THREADS, stream);
}

//    name, BM, BN, WM, WN, patch pixels, channel-fastest tensors
#define IGC_F32P_LIST(X) \
    X("f32 128x128x144 split patch", 128, 128, 2, 2, 384, false) \
    X("f32 128x128x144 split patch swap", 128, 128, 2, 2, 384, true) \
    X("f32 64x256x144 split patch", 64, 256, 1, 4, 512, false) \
    X("f32 64x256x144 split patch swap", 64, 256, 1, 4, 512, true) \
    X("f32 64x128x144 split patch", 64, 128, 2, 2, 640, false) \
    X("f32 64x128x144 split patch swap", 64, 128, 2, 2, 640, true)

#define IGC_F32P_INSTANTIATE(NAME, BM, BN, WM, WN, PIX, NHWC) \
    template __global__ void igconv_f32p_kernel<SplitPatchConfig<BM, BN, WM, WN, PIX, NHWC>>(const ConvKernelParams);
IGC_F32P_LIST(IGC_F32P_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
// (variant 5: operands split, patch)
#define IGC_F32P_ROW(NAME, BM, BN, WM, WN, PIX, NHWC)                                            \
    {NAME, false, BM, BN, 144, NHWC, false, 3, 512, SplitPatchConfig<BM, BN, WM, WN, PIX, NHWC>::LDS_BYTES, \
     &launch_f32p<SplitPatchConfig<BM, BN, WM, WN, PIX, NHWC>>, 5, false, PIX},
static const KernelInfo kRows[] = {IGC_F32P_LIST(IGC_F32P_ROW)};
const KernelGroup kGroupF32SplitPatch = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
