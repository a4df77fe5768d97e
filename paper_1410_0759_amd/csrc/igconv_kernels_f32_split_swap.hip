// fp32 kernels on the bfloat16 matrix pipes, every operand split into three parts (igconv_kernel_f32s.hpp): channel-fastest results
#include "igconv_instantiate.hpp"
#include "igconv_kernel_f32s.hpp"

namespace igc {

//    name, BM, BN, BK, WM, WN, swap, veca, window test, moving wavefronts, gather mode
#define IGC_F32S_LIST(X) \
    X("f32 64x128x32 split nopad swap", 64, 128, 32, 2, 2, true, false, false, 4, 2) \
    X("f32 64x128x32 split nopad swap vecw", 64, 128, 32, 2, 2, true, true, false, 4, 2) \
    X("f32 64x128x32 split border swap", 64, 128, 32, 2, 2, true, false, true, 4, 14) \
    X("f32 64x128x32 split border swap vecw", 64, 128, 32, 2, 2, true, true, true, 4, 14) \
    X("f32 128x128x32 split nopad swap", 128, 128, 32, 2, 2, true, false, false, 4, 2) \
    X("f32 128x128x32 split nopad swap vecw", 128, 128, 32, 2, 2, true, true, false, 4, 2) \
    X("f32 128x128x32 split border swap", 128, 128, 32, 2, 2, true, false, true, 4, 14) \
    X("f32 128x128x32 split border swap vecw", 128, 128, 32, 2, 2, true, true, true, 4, 14)

IGC_F32S_INSTANCES(kGroupF32SplitSwap)

}  // namespace igc
