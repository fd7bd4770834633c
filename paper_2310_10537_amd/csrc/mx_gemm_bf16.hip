// C = A B^T for bf16 operands [M][K] and [N][K] (K elements contiguous, K a multiple of 32), Float32 accumulation: what the MXINT8
// product runs on once its blocks have been multiplied by their scales (mx_gemm_int8.hip).  256 x 128 tiles for large whole ones
// (mx_gemm_bf16_half.hpp), else the tiles of mx_gemm_mid.hpp with the bf16 matrix instruction in place of the block-scaled one; to that
// kernel a row of 2K bytes looks like a row of 2K 8-bit elements.
#include "mx_gemm_bf16_half.hpp"
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
    const auto *A8 = static_cast<const uint8_t *>(A), *B8 = static_cast<const uint8_t *>(B);
    // columns c0 .. c0 + n - 1 of C on 128 x 128 tiles: three stages where one work-group per compute unit is all there is, two stages and
    // two work-groups otherwise
    auto mid = [&](int64_t c0, int64_t n) {
        const TileArgs a{M, n, 2 * K, A8, nullptr, nullptr, 0, ROUND_RNE, B8 + c0 * 2 * K, nullptr,
                         static_cast<uint8_t *>(C) + c0 * (c_dt == DT_F32 ? 4 : 2), c_dt, ldc, st};
        if (short_chains) return launch_mid_t<INT8, INT8, 2, 1, 3>(a);
        return ((M + 127) / 128) * ((n + 127) / 128) <= 256 ? launch_mid_t<INT8, INT8, 2, 2, 3>(a) : launch_mid_t<INT8, INT8, 2, 2, 2>(a);
    };
    if (short_chains) return mid(0, N);
    // 256 x 128 tiles where K is long enough for their start and end to be little (us, 128 x 128 / 256 x 128 in all: 8192 x 4096 x 512 61 / 62,
    // x 1024 90 / 91, x 2048 147 / 134, x 4096 269 / 236; 2048 x 3072 x 1024 32 / 32, x 2048 43 / 42; 8192^2 x 1024 157 / 162, x 2048 271 / 260), in
    // whole rounds of the 256 compute units or with a last round that is more than half full; the other columns go to 128 x 128 tiles
    // (4096 x 2816 x 4096, 352 tiles: 128 x 128 116, 256 x 128 114, 256 of them and 128 x 128 for the rest 105).
    const int64_t tiles_m = M / TM, tiles_n = N / HALF_N, tiles = tiles_m * tiles_n;
    int64_t cols = M % TM == 0 && N % HALF_N == 0 && K % 64 == 0 && K >= 2048 ? tiles_n : 0;
    if (tiles % 256 != 0 && tiles % 256 <= 128) cols = cols ? tiles / 256 * 256 / tiles_m : 0;
    if (cols == 0) return mid(0, N);
    const hipError_t e = c_dt == DT_F32 ? launch_bf16_half<DT_F32>(M, cols * HALF_N, K, A8, B8, C, ldc, st)
                                        : launch_bf16_half<DT_BF16>(M, cols * HALF_N, K, A8, B8, C, ldc, st);
    return e != hipSuccess || cols == tiles_n ? e : mid(cols * HALF_N, N - cols * HALF_N);
}

}  // namespace mx
