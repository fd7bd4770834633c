// MX GEMM that casts bf16 activations in registers, without scratch memory: the direct kernel of mx_gemm.hip on raw bf16 rows.
// Every 64-column tile of C casts its rows again, with the integer encoder, so this pays for short K only (see mx_gemm.hip);
// it also serves problems whose scratch memory was refused.
#include "mx_gemm_frag.hpp"
#include "mx_launch.hpp"

namespace mx {
namespace {

struct QaArgs {
    int64_t M, N, K;
    const void *a;
    int64_t lda;
    const uint8_t *Be, *Bs;
    void *C;
    int64_t ldc;
    hipStream_t st;
};

template <int FA, int FB, int RND, int CDT>
__global__ __launch_bounds__(256) void gemm_direct_qa_kernel(int64_t M, int64_t N, int64_t K, const uint16_t *__restrict__ A, int64_t lda,
                                                             const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                             void *__restrict__ C, int64_t ldc)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t m0 = (int64_t)blockIdx.y * 64 + (wave >> 1) * 32, n0 = (int64_t)blockIdx.x * 64 + (wave & 1) * 32;
    direct_tile<FA, FB, true, RND, CDT>(M, N, K, nullptr, nullptr, A, lda, Be, Bs, C, ldc, m0, n0, lane);
}

template <int FA, int FB, int RND, int CDT>
hipError_t go(const QaArgs &p)
{
    hipLaunchKernelGGL((gemm_direct_qa_kernel<FA, FB, RND, CDT>), dim3((unsigned)((p.N + 63) / 64), (unsigned)((p.M + 63) / 64)), dim3(256), 0,
                       p.st, p.M, p.N, p.K, static_cast<const uint16_t *>(p.a), p.lda, p.Be, p.Bs, p.C, p.ldc);
    return hipGetLastError();
}

template <int FA, int FB>
hipError_t pick(const QaArgs &p, int rnd, int c_dt)
{
    if (rnd == ROUND_RNE) return c_dt == DT_F32 ? go<FA, FB, ROUND_RNE, DT_F32>(p) : go<FA, FB, ROUND_RNE, DT_BF16>(p);
    return c_dt == DT_F32 ? go<FA, FB, ROUND_HALF_AWAY, DT_F32>(p) : go<FA, FB, ROUND_HALF_AWAY, DT_BF16>(p);
}

template <int FA>
hipError_t pick_b(const QaArgs &p, int fmtB, int rnd, int c_dt)
{
    switch (fmtB) {
        case FP8_E4M3: return pick<FA, FP8_E4M3>(p, rnd, c_dt);
        case FP8_E5M2: return pick<FA, FP8_E5M2>(p, rnd, c_dt);
        case FP6_E3M2: return pick<FA, FP6_E3M2>(p, rnd, c_dt);
        case FP6_E2M3: return pick<FA, FP6_E2M3>(p, rnd, c_dt);
        default:       return pick<FA, FP4_E2M1>(p, rnd, c_dt);
    }
}

}  // namespace

hipError_t launch_gemm_direct_qa(int64_t M, int64_t N, int64_t K, const void *a_bf16, int64_t lda, int rnd, int fmtA, const uint8_t *Be,
                                 const uint8_t *Bs, int fmtB, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    const QaArgs p{M, N, K, a_bf16, lda, Be, Bs, C, ldc, st};
    switch (fmtA) {
        case FP8_E4M3: return pick_b<FP8_E4M3>(p, fmtB, rnd, c_dt);
        case FP8_E5M2: return pick_b<FP8_E5M2>(p, fmtB, rnd, c_dt);
        case FP6_E3M2: return pick_b<FP6_E3M2>(p, fmtB, rnd, c_dt);
        case FP6_E2M3: return pick_b<FP6_E2M3>(p, fmtB, rnd, c_dt);
        default:       return pick_b<FP4_E2M1>(p, fmtB, rnd, c_dt);
    }
}

}  // namespace mx
