// LDS-tiled MX GEMM for any M, N and K of whole blocks, A operand FP4 (E2M1): every B format.
#include "mx_gemm_mid.hpp"

namespace mx {

hipError_t launch_gemm_mid_a4(const TileArgs &a, int fmtB) { return launch_mid_a<FP4_E2M1>(a, fmtB); }

}  // namespace mx
