// fp32 kernels on the bfloat16 matrix pipes, every operand split into three parts (igconv_kernel_f32s.hpp): no border
#include "igconv_instantiate.hpp"
#include "igconv_kernel_f32s.hpp"

namespace igc {

//    name, BM, BN, BK, WM, WN, swap, veca, window test, moving wavefronts, gather mode
#define IGC_F32S_LIST(X) \
    X("f32 64x128x32 split nopad", 64, 128, 32, 2, 2, false, false, false, 4, 2) \
    X("f32 64x128x32 split nopad vecw", 64, 128, 32, 2, 2, false, true, false, 4, 2) \
    X("f32 128x128x32 split nopad", 128, 128, 32, 2, 2, false, false, false, 4, 2) \
    X("f32 128x128x32 split nopad vecw", 128, 128, 32, 2, 2, false, true, false, 4, 2) \
    X("f32 96x128x32 split nopad", 96, 128, 32, 1, 4, false, false, false, 4, 2) \
    X("f32 96x128x32 split nopad vecw", 96, 128, 32, 1, 4, false, true, false, 4, 2) \

IGC_F32S_INSTANCES(kGroupF32SplitNopad)

}  // namespace igc
