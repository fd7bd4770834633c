// LDS-tiled MX GEMM for any M, N and K of whole blocks, A operand FP8 (E4M3 / E5M2); and the entry point.
#include "mx_gemm_mid.hpp"

namespace mx {

hipError_t launch_gemm_mid_a6(const TileArgs &a, int fmtA, int fmtB);
hipError_t launch_gemm_mid_a4(const TileArgs &a, int fmtB);

bool gemm_mid_applies(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    return fmtA >= FP8_E4M3 && fmtA <= FP4_E2M1 && fmtB >= FP8_E4M3 && fmtB <= FP4_E2M1 && M > 0 && N > 0 && K > 0 &&
           K <= (1 << 23) /* 32-bit byte offsets inside a tile */ && M <= (1 << 30) && N <= (1 << 30) &&
           ((M + 63) / 64) * ((N + 63) / 64) <= (1 << 24);
}

hipError_t launch_gemm_mid(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, int fmtA, const uint8_t *Be,
                           const uint8_t *Bs, int fmtB, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    if (!gemm_mid_applies(M, N, K, fmtA, fmtB)) return hipErrorNotSupported;
    const TileArgs a{M, N, K, Ae, As, nullptr, 0, ROUND_RNE, Be, Bs, C, c_dt, ldc, st};
    switch (fmtA) {
        case FP8_E4M3: return launch_mid_a<FP8_E4M3>(a, fmtB);
        case FP8_E5M2: return launch_mid_a<FP8_E5M2>(a, fmtB);
        case FP6_E3M2: case FP6_E2M3: return launch_gemm_mid_a6(a, fmtA, fmtB);
        default:       return launch_gemm_mid_a4(a, fmtB);
    }
}

}  // namespace mx
