// fp32 kernels on the bfloat16 matrix pipes, every operand split into three parts (igconv_kernel_f32s.hpp): any border
#include "igconv_instantiate.hpp"
#include "igconv_kernel_f32s.hpp"

namespace igc {

//    name, BM, BN, BK, WM, WN, swap, veca, window test, moving wavefronts, gather mode
#define IGC_F32S_LIST(X) \
    X("f32 64x128x32 split border", 64, 128, 32, 2, 2, false, false, true, 4, 14) \
    X("f32 64x128x32 split border vecw", 64, 128, 32, 2, 2, false, true, true, 4, 14) \
    X("f32 128x128x32 split border", 128, 128, 32, 2, 2, false, false, true, 4, 14) \
    X("f32 128x128x32 split border vecw", 128, 128, 32, 2, 2, false, true, true, 4, 14) \
    X("f32 96x128x32 split border", 96, 128, 32, 1, 4, false, false, true, 4, 14) \
    X("f32 96x128x32 split border vecw", 96, 128, 32, 1, 4, false, true, true, 4, 14)

IGC_F32S_INSTANCES(kGroupF32SplitBorder)

}  // namespace igc
