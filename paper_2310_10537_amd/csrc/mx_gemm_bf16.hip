// C = A B^T for bf16 operands [M][K] and [N][K] (K elements contiguous, K a multiple of 32), Float32 accumulation: what the MXINT8
// product runs on once its blocks have been multiplied by their scales (mx_gemm_int8.hip).  The tiles of mx_gemm_mid.hpp with the
// bf16 matrix instruction in place of the block-scaled one; to the kernel a row of 2K bytes looks like a row of 2K 8-bit elements.
//
// Bound by the cache lines that the tiles ask for (256 a step and work-group against 512 clocks of matrix instructions, 2.6 to 3.2
// clocks each).  256 x 256 tiles ask for half as many: 8192 x 4096 x 4096 219 us in all where 128 x 128 tiles take 277, but their
// accumulators leave no registers for sums of short chains, and the error of one chain over K is 3.4e-7 (2-norm, scales spread over 16
// octaves, K = 4096) where the E2M3 halves that this product replaced had 2.8e-7; 256 x 128 tiles with one wave per SIMD 301 us.
#include "mx_gemm_mid.hpp"

namespace mx {

bool gemm_bf16_applies(int64_t M, int64_t N, int64_t K)
{
    return M > 0 && N > 0 && K > 0 && K % BLOCK == 0 && K <= (1 << 21) /* 32-bit byte offsets inside a tile */ && M <= (1 << 30) &&
           N <= (1 << 30) && ((M + 63) / 64) * ((N + 63) / 64) <= (1 << 24);
}

hipError_t launch_gemm_bf16(int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, int c_dt, int64_t ldc,
                            bool short_chains, hipStream_t st)
{
    if (!gemm_bf16_applies(M, N, K)) return hipErrorNotSupported;
    const TileArgs a{M, N, 2 * K, static_cast<const uint8_t *>(A), nullptr, nullptr, 0, ROUND_RNE, static_cast<const uint8_t *>(B), nullptr,
                     C, c_dt, ldc, st};
    // Two sizes of tile, two depths of sums (mx_gemm_mid.hpp).  Three stages of a 128 x 128 tile where one work-group per compute unit is
    // all there is, two stages and two work-groups otherwise.
    if (short_chains) return launch_mid_t<INT8, INT8, 2, 1, 3>(a);
    return ((M + 127) / 128) * ((N + 127) / 128) <= 256 ? launch_mid_t<INT8, INT8, 2, 2, 3>(a) : launch_mid_t<INT8, INT8, 2, 2, 2>(a);
}

}  // namespace mx
