// bf16 kernels for any filter over channel-contiguous tensors, reading a filter rewritten with the channel index
// innermost (igconv_kernel_bf16_taps.hpp).
#include "igconv_instantiate.hpp"
#include "igconv_kernel_bf16_taps.hpp"

namespace igc {

template <class Cfg>
static int launch_taps(const ConvKernelParams &p, int grid, void *stream) {
    return launch_checked(&igconv_bf16_taps_kernel<Cfg>, "igconv_bf16_taps_kernel", p, grid, Cfg::THREADS, stream);
}

template <class Cfg>
static int launch_taps_phases(const ConvPhaseParams &p, int grid, void *stream) {
    return launch_checked(&igconv_bf16_taps_phases_kernel<Cfg>, "igconv_bf16_taps_phases_kernel", p, grid, Cfg::THREADS, stream);
}

#define IGC_TAPS_LIST(X)                                           \
    X("bf16 128x128x32 tapmajor vectors", 128, 128, 5, false)      \
    X("bf16 64x128x32 tapmajor vectors", 64, 128, 6, false)        \
    X("bf16 128x256x32 tapmajor vectors", 128, 256, 6, false)      \
    X("bf16 128x128x32 tapmajor vectors swap", 128, 128, 5, true)  \
    X("bf16 64x128x32 tapmajor vectors swap", 64, 128, 6, true)    \
    X("bf16 128x256x32 tapmajor vectors swap", 128, 256, 6, true)

#define IGC_TAPS_INSTANTIATE(NAME, BM, BN, STAGES, SWAP) \
    template __global__ void igconv_bf16_taps_kernel<Bf16TapsConfig<BM, BN, STAGES, SWAP>>(const ConvKernelParams); \
    template __global__ void igconv_bf16_taps_phases_kernel<Bf16TapsConfig<BM, BN, STAGES, SWAP>>(const ConvPhaseParams);
IGC_TAPS_LIST(IGC_TAPS_INSTANTIATE)

#if !defined(__HIP_DEVICE_COMPILE__)
#define IGC_TAPS_ROW(NAME, BM, BN, STAGES, SWAP) \
    {NAME, true, BM, BN, 32, SWAP, false, 1, Bf16TapsConfig<BM, BN, STAGES, SWAP>::THREADS, Bf16TapsConfig<BM, BN, STAGES, SWAP>::LDS_BYTES, \
     &launch_taps<Bf16TapsConfig<BM, BN, STAGES, SWAP>>, 6, false, 512, &launch_taps_phases<Bf16TapsConfig<BM, BN, STAGES, SWAP>>},
static const KernelInfo kRows[] = {IGC_TAPS_LIST(IGC_TAPS_ROW)};
const KernelGroup kGroupBF16Taps = {kRows, sizeof(kRows) / sizeof(kRows[0])};
#endif

}  // namespace igc
