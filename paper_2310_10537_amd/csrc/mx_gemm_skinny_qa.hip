// MX GEMM of up to 16 rows of bf16 activations that are cast on load (mx_gemm_skinny.hpp).
#include "mx_gemm_skinny.hpp"
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

template <int FA, int FB, int QA, int CDT>
hipError_t go(const QaArgs &p)
{
    hipLaunchKernelGGL((gemm_skinny_lds_kernel<FA, FB, 1, CDT, QA>), dim3((unsigned)((p.N + 31) / 32)), dim3(64 * SK_WAVES), 0, p.st, p.M, p.N,
                       p.K, static_cast<const uint8_t *>(p.a), (const uint8_t *)nullptr, p.Be, p.Bs, p.C, p.ldc, p.lda);
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

hipError_t launch_gemm_skinny_qa(int64_t M, int64_t N, int64_t K, const void *a_bf16, int64_t lda, int rnd, int fmtA, const uint8_t *Be,
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
