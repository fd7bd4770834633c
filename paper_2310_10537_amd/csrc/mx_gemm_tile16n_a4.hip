// 256 x 256 tiles on the 16 x 16 x 128 matrix instruction, A operand 4-bit, B operand 6-bit.
#include "mx_gemm_tile16n.hpp"

namespace mx {

hipError_t launch_gemm_tiled16n_a4(const TileArgs &a, int fmtA, int fmtB)
{
    (void)fmtA;
    return launch_a16n<FP4_E2M1>(a, fmtB);
}

}  // namespace mx
