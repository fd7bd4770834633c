// 256 x 256 tiles on the 16 x 16 x 128 matrix instruction, A operand 6-bit, B operand 6- or 4-bit.
#include "mx_gemm_tile16n.hpp"

namespace mx {

hipError_t launch_gemm_tiled16n_a6(const TileArgs &a, int fmtA, int fmtB)
{
    return fmtA == FP6_E3M2 ? launch_a16n<FP6_E3M2>(a, fmtB) : launch_a16n<FP6_E2M3>(a, fmtB);
}

}  // namespace mx
