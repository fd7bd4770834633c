// MX GEMM kernels (Section 4.1 of arXiv 2310.10537) on gfx950's block-scaled
// f8f6f4 matrix instruction:
//   C[m][n] = sum_b X_A[m][b] * X_B[n][b] * sum_j a[m][32b+j] * b[n][32b+j].
//
// V_MFMA_SCALE_F32_32X32X64_F8F6F4 register layout, established by one-hot and
// random-operand probes on the hardware (l = lane, i = l % 32, g = l / 32):
//   6- and 4-bit operands: lane l holds, for matrix row (A) / column (B) i, the
//     32 consecutive K elements [32g, 32g+32) densely bit-packed from bit 0
//     (FP6: 6 dwords, FP4: 4 dwords) -- one lane = one MX block;
//   8-bit operands: dwords 0-3 hold K [16g, 16g+16) and dwords 4-7 hold
//     K [32+16g, 32+16g+16), so a lane carries half of each of the two blocks;
//   scales: lane l supplies the E8M0 byte of row/column i, K block g (byte 0 of
//     the scale register with op_sel 0), whatever the element width;
//   result: lane l, register t holds C[8*(t/4) + 4*g + t%4][i].
// The kernel in this file uses the 32x32x64 form for every format pair.  Both forms run
// 6- and 4-bit pairs at twice the 8-bit rate and return the same bits; the 16x16x128 form, which
// needs less energy, is in the kernels for large products (mx_gemm_tile16.hpp, mx_gemm_tile16n.hpp).
#include "mx_gemm_frag.hpp"
#include "mx_launch.hpp"

namespace mx {

// ---------------------------------------------------------------------------
// Workspace of the routes that need scratch memory (see mx_launch.hpp)
// ---------------------------------------------------------------------------
namespace {
struct WsState { uint8_t *base; size_t bytes, used; bool active; };
thread_local WsState g_ws = {nullptr, 0, 0, false};
size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }
}  // namespace

WorkspaceScope::WorkspaceScope(void *p, size_t bytes) { g_ws = {static_cast<uint8_t *>(p), bytes, 0, p != nullptr}; }
WorkspaceScope::~WorkspaceScope() { g_ws = {nullptr, 0, 0, false}; }

hipError_t ws_acquire(size_t bytes, hipStream_t st, uint8_t **out)
{
    *out = nullptr;
    if (g_ws.active) {
        const size_t need = up256(bytes);
        if (g_ws.used + need > g_ws.bytes) return hipErrorOutOfMemory;
        *out = g_ws.base + g_ws.used;
        g_ws.used += need;
        return hipSuccess;
    }
    const hipError_t e = hipMallocAsync(reinterpret_cast<void **>(out), bytes, st);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

hipError_t ws_release(uint8_t *p, hipStream_t st)
{
    if (g_ws.active) {
        g_ws.used = (size_t)(p - g_ws.base);     // pieces are released in reverse order of acquisition
        return hipSuccess;
    }
    return hipFreeAsync(p, st);
}

static size_t cast_ws_bytes(int64_t M, int64_t K, int fmtA)
{
    const size_t bits = fmtA == FP4_E2M1 ? 4 : (fmtA == FP6_E3M2 || fmtA == FP6_E2M3) ? 6 : 8;
    return up256((size_t)M * (size_t)K * bits / 8 + 16) + up256((size_t)M * (size_t)(K / BLOCK));
}

size_t gemm_workspace_bound(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    return fmtA == INT8 && fmtB == INT8 ? gemm_int8_workspace(M, N, K) : 0;
}

size_t gemm_qa_workspace_bound(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    return cast_ws_bytes(M, K, fmtA) + gemm_workspace_bound(M, N, K, fmtA, fmtB);
}

size_t gemm_q_workspace_bound(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    if (M <= 0 || N <= 0) return 0;
    return up256((size_t)M * (size_t)((N + 3) & ~(int64_t)3) * sizeof(float)) + gemm_workspace_bound(M, N, K, fmtA, fmtB);
}

// ---------------------------------------------------------------------------
// Direct kernel: operands go from global memory straight into MFMA registers.
// Work-group = 4 waves, each wave one 32 x 32 output tile, K step 64.
// Handles every shape (ragged M, N; K any multiple of 32, K = 0 and K > 2^23 included).
// ---------------------------------------------------------------------------
template <int FA, int FB, int CDT>
__global__ __launch_bounds__(256) void gemm_direct_kernel(int64_t M, int64_t N, int64_t K,
                                                          const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                                          const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                          void *__restrict__ C, int64_t ldc)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t m0 = (int64_t)blockIdx.y * 64 + (wave >> 1) * 32;
    const int64_t n0 = (int64_t)blockIdx.x * 64 + (wave & 1) * 32;
    direct_tile<FA, FB, false, ROUND_RNE, CDT>(M, N, K, Ae, As, nullptr, 0, Be, Bs, C, ldc, m0, n0, lane);
}

struct GemmArgs {
    int64_t M, N, K;
    const uint8_t *Ae, *As, *Be, *Bs;
    void *C;
    int64_t ldc;
    hipStream_t st;
};

template <int FA, int FB, int CDT>
static hipError_t launch_direct(const GemmArgs &g)
{
    dim3 grid((unsigned)((g.N + 63) / 64), (unsigned)((g.M + 63) / 64));
    hipLaunchKernelGGL((gemm_direct_kernel<FA, FB, CDT>), grid, dim3(256), 0, g.st, g.M, g.N, g.K, g.Ae, g.As, g.Be, g.Bs, g.C, g.ldc);
    return hipGetLastError();
}

template <int FA>
static hipError_t dispatch_b(const GemmArgs &g, int fmtB, int c_dt)
{
#define MX_GO(FB) (c_dt == DT_F32 ? launch_direct<FA, FB, DT_F32>(g) : launch_direct<FA, FB, DT_BF16>(g))
    switch (fmtB) {
        case FP8_E4M3: return MX_GO(FP8_E4M3);
        case FP8_E5M2: return MX_GO(FP8_E5M2);
        case FP6_E3M2: return MX_GO(FP6_E3M2);
        case FP6_E2M3: return MX_GO(FP6_E2M3);
        default:       return MX_GO(FP4_E2M1);
    }
#undef MX_GO
}

// How a product of FP8 / FP6 / FP4 operands is computed; the choice depends on the shape and the formats only.
enum Route {
    SHARED_K,    // eight waves share the K range of 32 columns (mx_gemm_skinny.hip): few rows, or too few tiles to fill the chip
    MID,         // 64 x 64 to 128 x 128 tiles (mx_gemm_mid.hpp): any shape
    WHOLE,       // 256 x 256 tiles (mx_gemm_tile*.hpp), nothing left over
    INTERIOR,    // 256 x 256 tiles over the largest interior they cover, MID for the L-shaped fringe
    DIRECT       // short K, and what none of the others takes: K = 0; K beyond 2^23 and no multiple of 128, more than 128 rows
};

// Beyond the MID kernel's sizes (K over 2^23, over 2^24 tiles of 64 x 64): up to 128 rows SHARED_K, then 256 x 256 tiles, then
// SHARED_K in groups of 128 rows.  A long K needs the waves: the direct kernel walks all of it with one wave per 32 x 32 tile.
// Measured boundaries (E4M3 pairs unless said otherwise; us):
//  - DIRECT for short K, more than 64 rows: a tile's load, wait, multiply and store take their time however few steps lie between.
//    MID / DIRECT: 593 x 7040 x 64 10.6 / 5.9, 8192 x 8192 x 64 64 / 43, 1536 x 8704 x 128 19 / 19 and E3M2 20 / 12,
//    8192 x 8192 x 128 61 / 77 and E3M2 61 / 50, 8192 x 8192 x 192 81 / 73, 1536 x 8704 x 256 21 / 31. Narrow operands load less per step, and
//    the line moves on: E3M2 593 x 7040 x 384 13 / 12, 4096 x 1536 x 384 14 / 16; E4M3 x E2M1 1000 x 1000 x 256 5.3 / 5, 593 x 7040
//    level, 1536 x 8704 21 / 26; a partial last step, E4M3 768 x 2560 x 288 7.0 / 6.0, with E2M1 593 x 7040 x 288 10.5 / 9.0.
//  - SHARED_K or MID.  Up to 32 rows the weight stream decides and the shared-K kernel reads it best; 33 to 64 rows: 64 x 1024 x 4096
//    level, 64 x 4096 x 4096 16 against 11, 64 x 11008 x 4096 31 against 15.  Above 64 rows the shared-K kernel holds
//    so many accumulators that one work-group fills a compute unit: 128 x 1024 x 4096 22 against 11, 256 x 4096 x 4096 25 against
//    12 -- but a handful of tiles with a short K stays with it.
//  - MID or 256 x 256 tiles.  2048^3 (64 whole tiles, one 128 x 128 tile per compute unit) 19 against 15, E2M1 15 against 12;
//    2048 x 4096 x 4096 (128) 41 against 42, E3M2 x E2M1 36 against 40; 4096^3 (256) 61 against 85.
//  - A problem with a fringe costs an extra launch or two that each leave most of the chip idle: 1000 x 4096 x 4096 60 against 26,
//    5000 x 11008 x 4096 (817 whole tiles) 280 against 291; the line in between: interior_pays.
static bool direct_pays(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    if (M <= 64 || (M + 63) / 64 > 65535) return false;                     // (the direct kernel's grid)
    const int narrow = (fmt_bits(fmtA) < 8) + (fmt_bits(fmtB) < 8);
    if (K < 256) return !(narrow == 0 && K == 128 && M * N > ((int64_t)1 << 24));
    const bool tail = K % 128 != 0;                                          // one more, partial step in the MID kernel
    return K < 512 && M * N * K <= (narrow == 2 ? (int64_t)1 << 31 : narrow == 1 ? (int64_t)(tail ? 3 : 1) << 29 : (int64_t)(tail ? 5 : 0) << 27);
}

// Whether an interior of 129 to 192 whole tiles with a fringe goes to 256 x 256 tiles: one or two more launches against a K loop that
// runs at two thirds of the rate or less, so the longer K the better, and the sooner the narrower the operands of both sides.
// MID / INTERIOR, us: fringe on one side, 3100 x 3072 x 4096 E4M3 59 / 54, E3M2 58 / 46, E3M2 x E2M1 49 / 39, E4M3 x E2M1 47 / 51; K = 2048
// 33 / 34, 33 / 28, 28 / 25; E3M2 K = 1024 22 / 20; on both sides, 3340 x 3340 x 4096 65 / 62, 69 / 59, 53 / 52, 49 / 62, K = 8192 122 / 110,
// 129 / 104, 97 / 91, 92 / 107.  Interiors of 100 tiles: MID is ahead (2600 x 2560 x 4096 E4M3 34 / 43) but for 6-bit pairs (40 / 40; K = 8192 76 / 69).
// A very long K moves the line further: 1568 x 3584 (84 tiles) x 8192 E3M2 79 / 66, E2M1 x E3M2 68 / 54, x 16384 E2M1 92 / 83, E5M2 x E2M3 x 24960
// 147 / 139.
static bool interior_pays(int64_t M, int64_t N, int64_t K, int64_t whole, int fmtA, int fmtB)
{
    if (whole > 192) return true;
    const int a = fmt_bits(fmtA), b = fmt_bits(fmtB);
    const bool both = M % 256 != 0 && N % 256 != 0;
    if (a + b == 12 && a != b) return !both && whole > 184 && K >= 4096;      // 8 x 4 bits
    if (whole > 72 && !both && a < 8 && b < 8 && (K >= 16384 || (K >= 8192 && b == 6))) return true;
    if (whole <= (a + b == 12 && !both && K >= 4096 ? 96 : 128)) return false;
    if (both) return K >= (a + b == 12 || a + b == 10 ? 4096 : 6144);
    return K >= (a + b == 16 ? 4096 : a + b == 12 ? 1024 : 2048);
}

static Route route_of(int64_t M, int64_t N, int64_t K, int fmtA, int fmtB)
{
    const int64_t M0 = M & ~(int64_t)255, N0 = N & ~(int64_t)255;
    const bool shared_ok = gemm_skinny_applies(M, N, K, fmtA, fmtB);
    if (!gemm_mid_applies(M, N, K, fmtA, fmtB)) {
        if (shared_ok && M <= 128) return SHARED_K;
        if (gemm_tiled_applies(M0, N0, K, fmtA, fmtB)) return M0 == M && N0 == N ? WHOLE : INTERIOR;
        return shared_ok ? SHARED_K : DIRECT;
    }
    const int64_t tiles64 = ((M + 63) / 64) * ((N + 63) / 64);
    const bool shared = M <= 32 || (M <= 64 ? tiles64 < 64 : tiles64 < 24 && K < 4096);
    if (shared && shared_ok) return SHARED_K;
    if (direct_pays(M, N, K, fmtA, fmtB)) return DIRECT;
    const int64_t whole = (M0 / 256) * (N0 / 256);
    if (M0 == M && N0 == N) return whole > 64 && gemm_tiled_applies(M, N, K, fmtA, fmtB) ? WHOLE : MID;
    return interior_pays(M, N, K, whole, fmtA, fmtB) && gemm_tiled_applies(M0, N0, K, fmtA, fmtB) ? INTERIOR : MID;
}

// whether the fused quantize-on-load tiled kernel beats cast + plain tiled kernel (256 x 256 tiles)
static bool qa_fused_pays(int64_t M, int64_t N) { return N / 256 <= 2 && (M / 256) * (N / 256) >= 256; }

// Whether the shared-K kernel casts few rows on load: every work-group casts its slice again (16 rows: a block a lane), mostly behind
// the weight stream, against a launch and a stream-ordered workspace.  bf16 out, cast apart -> on load: 1 x 4096 x 4096 E4M3 27.9 ->
// 9.1 us, 1 x 11008 x 4096 28.2 -> 11.7, 16 x 11008 x 4096 29.0 -> 13.7, 16 x 28672 x 8192 68.3 -> 63.4, E3M2 x E2M1 46.7 -> 41.9.
static bool qa_few_rows_pays(int64_t M, int64_t K) { return M <= 16 && K % 128 == 0; }

// Whether A can do without scratch memory where the few-rows kernel does not cast it: more than 128 rows with K below 512 or no multiple
// of 128, round to nearest.  Such problems are cast in registers when that is faster, and when scratch memory is refused.
static bool qa_in_registers(int64_t M, int64_t K, int rnd)
{
    return M > 128 && (M + 63) / 64 <= 65535 && (K % 128 != 0 || K < 512) && (rnd == ROUND_RNE || rnd == ROUND_HALF_AWAY);
}

// The cast in registers takes about 4 + K (0.018 + 0.024 w) us, w = M N / 2^20 waves of a SIMD (at least one): 300 x 500 x 160 9.8,
// 768 x 2560 x 288 21, 1000 x 4096 x 128 19, 4096 x 1536 x 96 24 (E4M3; a seventh less below 8 bits).  Cast and product apart take
// about 9 us when these times are short, and 21 with a stream-ordered allocation and its release.
static bool qa_in_registers_pays(int64_t M, int64_t N, int64_t K, int fmtA, bool own_scratch)
{
    const int64_t w16 = M * N >> 16;                                        // sixteenths of w
    return K * (18 + 24 * (w16 > 16 ? w16 : 16) / 16) < (own_scratch ? 4000 : fmt_bits(fmtA) < 8 ? 20000 : 17000);
}

static size_t mx_bytes16(int64_t M, int64_t K, int fmt) { return ((size_t)M * (size_t)K * fmt_bits(fmt) / 8 + 15) & ~(size_t)15; }

// A problem whose M or N is not a multiple of the 256 x 256 tile may be cut into the largest interior of whole tiles and an L-shaped
// fringe of fewer than 256 rows / columns.  Every output entry is computed by exactly one launch; which one
// depends on the shape only, so a result is reproducible, and quantize-on-load follows the same cut.
hipError_t launch_gemm(int64_t M, int64_t N, int64_t K, const uint8_t *A_elems, const uint8_t *A_scales,
                       const void *a_bf16, int64_t lda, int rnd, int fmtA, const uint8_t *B_elems,
                       const uint8_t *B_scales, int fmtB, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    const bool int8 = fmtA == INT8 && fmtB == INT8;
    const int64_t M0 = M & ~(int64_t)255, N0 = N & ~(int64_t)255;
    const Route route = int8 ? DIRECT : route_of(M, N, K, fmtA, fmtB);
    // Quantize-on-load.  The fused tiled kernel casts each A tile once per column of output tiles and reads it as bf16 that
    // often, so it pays only for narrow outputs (measured: up to two tile columns), and only when there are enough tiles to
    // fill the chip, since the stand-alone cast always runs on every compute unit.  Up to 16 rows are cast by the
    // shared-K kernel, a short K in registers by the direct one.  Every other problem casts A once
    // into a workspace (the same cast kernel, hence the same bytes, as mx_quantize) and runs the plain product on it.
    const bool fused = a_bf16 && (rnd == ROUND_RNE || rnd == ROUND_HALF_AWAY) && (route == WHOLE || route == INTERIOR) &&
                       gemm_tiled_fuses_cast(fmtA, fmtB) && qa_fused_pays(M0, N0);
    if (a_bf16 && route == SHARED_K && qa_few_rows_pays(M, K) && (rnd == ROUND_RNE || rnd == ROUND_HALF_AWAY))
        return launch_gemm_skinny_qa(M, N, K, a_bf16, lda, rnd, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
    if (a_bf16 && !fused && M > 0 && N > 0 && K > 0) {
        const bool registers = !int8 && qa_in_registers(M, K, rnd);
        auto in_registers = [&]() { return launch_gemm_direct_qa(M, N, K, a_bf16, lda, rnd, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st); };
        if (registers && qa_in_registers_pays(M, N, K, fmtA, g_ws.active)) return in_registers();
        const size_t eb = mx_bytes16(M, K, fmtA), sb = (size_t)M * (size_t)(K / BLOCK);
        uint8_t *ws = nullptr;
        hipError_t e = ws_acquire(eb + sb, st, &ws);
        if (e != hipSuccess) return registers ? in_registers() : e;
        e = launch_cast(a_bf16, DT_BF16, M, K, lda, 1, fmtA, rnd, ws, ws + eb, st);
        if (e == hipSuccess)
            e = launch_gemm(M, N, K, ws, ws + eb, nullptr, 0, ROUND_RNE, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
        const hipError_t f = ws_release(ws, st);
        return e != hipSuccess ? e : f;
    }
    if (int8) return launch_gemm_int8(M, N, K, A_elems, A_scales, B_elems, B_scales, C, c_dt, ldc, st);
    switch (route) {
        case SHARED_K: return launch_gemm_skinny(M, N, K, A_elems, A_scales, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
        case MID:      return launch_gemm_mid(M, N, K, A_elems, A_scales, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
        case WHOLE:
            return launch_gemm_tiled(M, N, K, A_elems, A_scales, a_bf16, lda, rnd, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
        case DIRECT: {
            const GemmArgs g{M, N, K, A_elems, A_scales, B_elems, B_scales, C, ldc, st};
            switch (fmtA) {
                case FP8_E4M3: return dispatch_b<FP8_E4M3>(g, fmtB, c_dt);
                case FP8_E5M2: return dispatch_b<FP8_E5M2>(g, fmtB, c_dt);
                case FP6_E3M2: return dispatch_b<FP6_E3M2>(g, fmtB, c_dt);
                case FP6_E2M3: return dispatch_b<FP6_E2M3>(g, fmtB, c_dt);
                default:       return dispatch_b<FP4_E2M1>(g, fmtB, c_dt);
            }
        }
        default: break;
    }
    const int64_t bitsA = fmt_bits(fmtA), bitsB = fmt_bits(fmtB), nkb = K / BLOCK, esz = c_dt == DT_F32 ? 4 : 2;
    const uint8_t *a16 = static_cast<const uint8_t *>(a_bf16);
    uint8_t *c8 = static_cast<uint8_t *>(C);
    hipError_t e = launch_gemm_tiled(M0, N0, K, A_elems, A_scales, a_bf16, lda, rnd, fmtA, B_elems, B_scales, fmtB, C, c_dt, ldc, st);
    auto fringe = [&](int64_t r0, int64_t rows, int64_t c0, int64_t cols) {
        return launch_gemm(rows, cols, K, A_elems ? A_elems + r0 * (K * bitsA / 8) : nullptr, A_scales ? A_scales + r0 * nkb : nullptr,
                           a16 ? a16 + r0 * lda * 2 : nullptr, lda, rnd, fmtA, B_elems + c0 * (K * bitsB / 8), B_scales + c0 * nkb, fmtB,
                           c8 + (r0 * ldc + c0) * esz, c_dt, ldc, st);
    };
    if (e == hipSuccess && M > M0) e = fringe(M0, M - M0, 0, N);
    if (e == hipSuccess && N > N0) e = fringe(0, M0, N0, N - N0);
    return e;
}

// C as an MX tensor.  Whole-tile problems cast the accumulators in the tiled kernel's epilogue;
// every other problem (MXINT8 operands, truncated output) writes C as Float32 into a stream-ordered
// workspace and casts that -- the same accumulators and the same Algorithm 1, hence the same bytes.
hipError_t launch_gemm_q(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, int fmtA, const uint8_t *Be,
                         const uint8_t *Bs, int fmtB, uint8_t *Ce, uint8_t *Cs, int fmtC, int rndC, hipStream_t st)
{
    // The tiled kernel's accumulators are those of mx_gemm on every route but SHARED_K.  Below 32 tiles (44 with a long K) it would
    // leave most of the chip idle for longer than writing and casting a Float32 C takes.
    const int64_t tiles = (M / 256) * (N / 256);
    if (fmtA != INT8 && tiles >= 32 && (tiles >= 44 || K < 8192) && route_of(M, N, K, fmtA, fmtB) != SHARED_K) {
        const hipError_t e = launch_gemm_tiled_mx(M, N, K, Ae, As, fmtA, Be, Bs, fmtB, Ce, Cs, fmtC, rndC, st);
        if (e != hipErrorNotSupported) return e;
    }
    float *ws = nullptr;
    const int64_t ldw = (N + 3) & ~(int64_t)3;   // rows of the workspace stay 16-byte aligned
    uint8_t *ws8 = nullptr;
    hipError_t e = ws_acquire((size_t)M * (size_t)ldw * sizeof(float), st, &ws8);
    if (e != hipSuccess) return e;
    ws = reinterpret_cast<float *>(ws8);
    e = launch_gemm(M, N, K, Ae, As, nullptr, 0, ROUND_RNE, fmtA, Be, Bs, fmtB, ws, DT_F32, ldw, st);
    if (e == hipSuccess) e = launch_cast(ws, DT_F32, M, N, ldw, 1, fmtC, rndC, Ce, Cs, st);
    const hipError_t f = ws_release(ws8, st);
    return e != hipSuccess ? e : f;
}

}  // namespace mx
