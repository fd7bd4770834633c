// C = A B^T for bf16 operands on 256 x 128 tiles (see mx_gemm_bf16.hip): whole tiles, K a multiple of 64, Float32 accumulation in two
// halves of K.
//
// Work-group: four waves of 128 x 64, i.e. 8 x 4 tiles of the 16 x 16 x 32 instruction, K step 64 (128 bytes of a row, two instructions a
// tile).  LDS layout, direct loads and operand reads as in mx_gemm_tile16.hpp; the fragments of a step's rows 0-63 and of its columns
// are read in the step before, those of rows 64-127 beside the first half of its instructions; one barrier stands between the halves,
// behind which the stage three steps on is requested, in three stages of 48 KB: a third of its loads at once, the others beside the first
// half of the next step, where there are fewer operand reads (all at once 1 to 2 % slower).
//
// Bound by the LDS: 96 KB of operand reads and 48 KB of direct loads a step are 1152 of its clocks against 1024 of the matrix pipe, and by
// the energy limit.  8192 x 4096 x 4096 in all: 233 us, 128 x 128 tiles 263, 256 x 256 tiles 209.
//
// Why this tile.  256 x 256 tiles keep 256 accumulators a lane and have no registers for more, and one chain of the bf16 instruction over
// all of K errs by 3.4e-7 (2-norm, scales of MXINT8 blocks spread over 16 octaves, K = 4096), where the product on E2M3 halves that this one
// stands for had 2.8e-7.  With 128 accumulators the sum of the first half of K is set aside and the second begins at zero: 2.4e-7.
#pragma once
#include "mx_gemm_tile16.hpp"

namespace mx {

typedef int int32x4_t __attribute__((ext_vector_type(4)));

// The accumulator is updated in place in the accumulation registers, as in mfma16
__device__ __forceinline__ void mfma16_bf16(v4f_t &acc, const int32x4_t &op1, const int32x4_t &op2)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(op1), "v"(op2));
}

constexpr int HALF_N = 128;

template <int CDT>
__global__ __launch_bounds__(256, 1) void gemm_bf16_half_kernel(int64_t K, const uint8_t *__restrict__ A, const uint8_t *__restrict__ B,
                                                                void *__restrict__ C, int64_t ldc, int tiles_m, int tiles_n, Raster rast)
{
    constexpr int STEP = 128;                                  // bytes of a row
    constexpr int A_BYTES = TM * STEP, STAGE_BYTES = (TM + HALF_N) * STEP;
    constexpr int NJA = A_BYTES / 4096, NJ = STAGE_BYTES / 4096;       // direct loads per wave and stage (1 KB each): 8 of A, 4 of B
    constexpr int FIRST = 4;                                   // ... that go out right behind the barrier
    __shared__ __attribute__((aligned(16))) uint8_t lds[3 * STAGE_BYTES];
    static_assert(sizeof(lds) <= 160 * 1024, "LDS of a compute unit");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, i = lane & 15, q = lane >> 4;

    int tm, tn;
    if (!raster_tile(rast, (int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * HALF_N;
    const int64_t row = 2 * K;
    const int T = (int)(row / STEP);                           // K steps
    const int T1 = (T / 2) & ~1;                               // ... of the first half, an even number

    // wave w, load j of an operand's tile: rows (4j + w) * 8 .. + 7, lane l into slot l % 8 of row l / 8 of them
    const int s_r = lane >> 3, s_u = (lane & 7) ^ (((wave * 8 + s_r) >> 1) & 7);
    const uint8_t *gA = A + (m0 + wave * 8 + s_r) * row + s_u * 16;
    const uint8_t *gB = B + (n0 + wave * 8 + s_r) * row + s_u * 16;
    typedef __attribute__((address_space(3))) void lds_ptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t *)lds) + wave * 1024;
    // direct load k of step t (A's, then B's) into the stage at byte offset dst; beyond the end the last step again, never read
    auto stage_one = [&](int k, int t, int dst) __attribute__((always_inline)) {
        t = t < T ? t : T - 1;
        const uint8_t *gp = (k < NJA ? gA + k * 32 * row : gB + (k - NJA) * 32 * row) + (int64_t)t * STEP;
        asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(gp), "s"(lds0 + dst + k * 4096) : "m0", "memory");
    };
    // operand reads: tile row wm*128 + 16x + i (A) / wn*64 + 16y + i (B), chunks q and q + 4: the first and the second 32 elements
    const int ra = (wm * 128 + i) * STEP + ((q ^ ((i >> 1) & 7)) << 4);
    const int rb = A_BYTES + (wn * 64 + i) * STEP + ((q ^ ((i >> 1) & 7)) << 4);
    struct Frag { int32x4_t lo, hi; };
    auto frag = [&](Frag &f, int ofs, int xb) __attribute__((always_inline)) {
        f.lo = *reinterpret_cast<const int32x4_t *>(lds + ofs + xb * 2048);
        f.hi = *reinterpret_cast<const int32x4_t *>(lds + (ofs ^ 64) + xb * 2048);
    };

    v4f_t acc[8][4], sum[8][4];
#pragma unroll
    for (int x = 0; x < 8; x++)
#pragma unroll
        for (int y = 0; y < 4; y++) { acc[x][y] = v4f_t{0.f, 0.f, 0.f, 0.f}; sum[x][y] = acc[x][y]; }
    Frag aL[4], aH[4], bE[4], bO[4];

#pragma unroll
    for (int s = 0; s < 3; s++)
#pragma unroll
        for (int k = 0; k < (s < 2 ? NJ : FIRST); k++) stage_one(k, s, s * STAGE_BYTES);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NJ + FIRST) : "memory");
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 4; x++) { frag(aL[x], ra, x); frag(bE[x], rb, x); }
    int cur = 0, nxt = STAGE_BYTES, aft = 2 * STAGE_BYTES;      // stages of steps t, t + 1, t + 2

#define MX_FENCE() __builtin_amdgcn_sched_barrier(0)
    // column tile y: the two instructions of four row tiles each, X0 .. X0 + 3; `slot` stands in front of every second one
    auto column = [&](auto &AS, const Frag &b, const int X0, const int y, auto &&slot) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 8; m++) {
            if ((m & 1) == 0) slot(m / 2);
            const int x = m & 3;
            if (m < 4) mfma16_bf16(acc[X0 + x][y], b.lo, AS[x].lo);
            else mfma16_bf16(acc[X0 + x][y], b.hi, AS[x].hi);
            if (m & 1) MX_FENCE();
        }
    };
    auto step = [&](Frag (&b)[4], Frag (&bn)[4], const int t) __attribute__((always_inline)) {
        MX_FENCE();
#pragma unroll
        for (int y = 0; y < 4; y++)
            column(aL, b[y], 0, y, [&](int s) __attribute__((always_inline)) {
                if (s & 1) stage_one(FIRST + 2 * y + s / 2, t + 2, aft);
                if (y == 0 && (s == 0 || s == 2)) frag(aH[s / 2], cur + ra, 4 + s / 2);
                if ((y == 1 || y == 2) && s == 0) frag(aH[1 + y], cur + ra, 5 + y);
            });
        // step t + 1 must be in LDS -- step t + 2, requested since the last barrier, may be in flight -- and every wave must have read its
        // operands of step t, before the stage takes step t + 3
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NJ) : "memory");
        __syncthreads();
        MX_FENCE();
#pragma unroll
        for (int y = 0; y < 4; y++)
            column(aH, b[y], 4, y, [&](int s) __attribute__((always_inline)) {
                if (s == 3) stage_one(y, t + 3, cur);
                if (y < 2 && s < 2) frag(aL[2 * y + s], nxt + ra, 2 * y + s);
                if (y < 2 && s == 2) frag(bn[y], nxt + rb, y);
                if (y == 2 && s < 2) frag(bn[2 + s], nxt + rb, 2 + s);
            });
        const int was = cur;
        cur = nxt; nxt = aft; aft = was;
        MX_FENCE();
    };
    // Behind the last matrix instruction: the compiler, which takes the assembly for something else, leaves no wait states
    auto settle = [&]() __attribute__((always_inline)) {
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
        for (int x = 0; x < 8; x++) asm volatile("" : "+a"(acc[x][0]), "+a"(acc[x][1]), "+a"(acc[x][2]), "+a"(acc[x][3]));
    };
    for (int t = 0; t < T1; t += 2) {
        step(bE, bO, t);
        step(bO, bE, t + 1);
    }
    settle();
#pragma unroll
    for (int x = 0; x < 8; x++)
#pragma unroll
        for (int y = 0; y < 4; y++) { sum[x][y] = acc[x][y]; acc[x][y] = v4f_t{0.f, 0.f, 0.f, 0.f}; }
    MX_FENCE();
    asm volatile("s_nop 7" ::: "memory");                     // vector writes of accumulators -> matrix instruction
    for (int t = T1; t + 1 < T; t += 2) {
        step(bE, bO, t);
        step(bO, bE, t + 1);
    }
    if (T & 1) step(bE, bO, T - 1);
#undef MX_FENCE
    settle();
#pragma unroll
    for (int x = 0; x < 8; x++)
#pragma unroll
        for (int y = 0; y < 4; y++) acc[x][y] += sum[x][y];
    store_tile16<CDT>(acc, C, ldc, m0 + wm * 128, n0 + wn * 64, i, q);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // requests past the end have landed before the LDS is given up
}

template <int CDT>
static hipError_t launch_bf16_half(int64_t M, int64_t N, int64_t K, const uint8_t *A, const uint8_t *B, void *C, int64_t ldc, hipStream_t st)
{
    const int tiles_m = (int)(M / TM), tiles_n = (int)(N / HALF_N);
    const Raster rast = choose_raster(tiles_m, tiles_n, 8, 8);
    hipLaunchKernelGGL((gemm_bf16_half_kernel<CDT>), dim3(raster_grid(rast, tiles_m, tiles_n)), dim3(256), 0, st, K, A, B, C, ldc, tiles_m,
                       tiles_n, rast);
    return hipGetLastError();
}

}  // namespace mx
