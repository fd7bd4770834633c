// C = A B^T for bf16 operands [M][K] and [N][K] (K elements contiguous, K a multiple of 32), Float32 accumulation: what the MXINT8
// product runs on once its blocks have been multiplied by their scales (mx_gemm_int8.hip).  The 256 x 256 tiles of
// mx_gemm_tile16.hpp and the smaller ones of mx_gemm_mid.hpp with the bf16 matrix instructions in place of the block-scaled ones; to
// both a row of 2K bytes looks like a row of 2K 8-bit elements.
#include "mx_gemm_mid.hpp"
#include "mx_gemm_tile16.hpp"

namespace mx {

bool gemm_bf16_applies(int64_t M, int64_t N, int64_t K)
{
    return M > 0 && N > 0 && K > 0 && K % BLOCK == 0 && K <= (1 << 22) /* 32-bit byte offsets inside a tile */ && M <= (1 << 30) &&
           N <= (1 << 30) && ((M + 63) / 64) * ((N + 63) / 64) <= (1 << 24);
}

static hipError_t bf16_mid(const TileArgs &a) { return launch_mid_pair<INT8, INT8>(a); }

static hipError_t bf16_whole(const TileArgs &a)
{
    return a.c_dt == DT_F32 ? launch_t16<INT8, INT8, DT_F32>(a.M, a.N, a.K, a.Ae, a.As, a.Be, a.Bs, a.C, a.ldc, a.st)
                            : launch_t16<INT8, INT8, DT_BF16>(a.M, a.N, a.K, a.Ae, a.As, a.Be, a.Bs, a.C, a.ldc, a.st);
}

hipError_t launch_gemm_bf16(int64_t M, int64_t N, int64_t K, const void *A, const void *B, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    if (!gemm_bf16_applies(M, N, K)) return hipErrorNotSupported;
    const auto *A8 = static_cast<const uint8_t *>(A), *B8 = static_cast<const uint8_t *>(B);
    const int64_t esz = c_dt == DT_F32 ? 4 : 2;
    // rows r0 .. r0 + m - 1 and columns c0 .. c0 + n - 1 of C
    auto part = [&](bool whole, int64_t r0, int64_t m, int64_t c0, int64_t n) {
        if (m <= 0 || n <= 0) return hipSuccess;
        const TileArgs a{m, n, 2 * K, A8 + r0 * 2 * K, nullptr, nullptr, 0, ROUND_RNE, B8 + c0 * 2 * K, nullptr,
                         static_cast<uint8_t *>(C) + (r0 * ldc + c0) * esz, c_dt, ldc, st};
        return whole ? bf16_whole(a) : bf16_mid(a);
    };
    // As many columns of 256 x 256 tiles as make up whole rounds of the 256 compute units (all of them where the last round is more
    // than half full), the smaller tiles for the rest.
    const int64_t tiles_m = M / TM, tiles_n = N / TN, tiles = tiles_m * tiles_n;
    int64_t cols = tiles_n;
    if (tiles % 256 != 0 && tiles % 256 <= 128) cols = tiles_m > 0 ? tiles / 256 * 256 / tiles_m : 0;
    if (K % 64 != 0 || tiles_m * cols <= 128) cols = 0;
    const int64_t m0 = cols ? tiles_m * TM : 0, n0 = cols * TN;
    hipError_t e = part(true, 0, m0, 0, n0);
    if (e == hipSuccess) e = part(false, m0, M - m0, 0, cols ? n0 : N);          // below the whole tiles, or everything
    if (e == hipSuccess && cols) e = part(false, 0, M, n0, N - n0);               // right of them
    return e;
}

}  // namespace mx
