// LDS-tiled MX GEMM (Section 4.1 of arXiv 2310.10537) for pairs of 6- and 4-bit formats on the 16 x 16 x 128 form of the
// block-scaled matrix instruction: 256 x 256 tile, K step 128, four waves of 128 x 128 (8 x 8 instructions a step), whole tiles,
// K a multiple of 512, plain operands, Float32 / bf16 output.
//
// The instruction.  For 6- and 4-bit operands it issues every 17.8 clocks for the work that the 32 x 32 x 64 form does in 16, and
// needs less energy for it: from registers, on random codes, 5.6 against 5.2 PFLOP/s (E3M2) and 6.7 against 6.1 (E2M1) at the
// board's power limit.  Lane l, i = l % 16, q = l / 16 holds the 32 elements of block q of row i, densely packed; the scale byte is
// that block's; result register t is D[4q + t][i].  One instruction returns the bits of two chained 32 x 32 x 64 instructions
// (compared on the GPU for every pair of formats, with random scales and accumulator inputs: 2 million entries each, none
// different), so every kernel for these pairs gives the same bits.  A fragment is 16 whole 96-byte rows of the tile, which 8-byte reads
// cover at 2.6 LDS clocks each; 32 rows at a 96-byte pitch took 4 (two rows per bank pair).
//
// The loads.  What bounds a K step is not the matrix pipe (64 x 17.8 = 1140 clocks) and not the bytes, but the cache lines that a
// compute unit asks for: 2.6 to 3.2 clocks each, whole or not.  A step's 96 (64) bytes of a row are parts of one or two lines, every one
// of which is asked for again in the next step: 44 clocks per KB loaded and 2350 clocks a step on zeros, with direct loads to LDS
// for each step.  Here a load fetches whole lines, eight rows of 128 bytes: 26 clocks per KB.  Three lines are four steps of a 6-bit
// row, two of a 4-bit row, and there is no LDS for them to wait in (three stages of one step each fill it), so they wait in
// registers, 16 bytes a lane for each of 16 loads, and are written to the one or two stages they belong to when those are free: the
// window behind the barrier of step t for the steps t + 2 and t + 3.  Lines of 8 rows go out as two pieces of 64 bytes of two rows
// after the other, so that the 8 lanes of an LDS write phase meet no bank twice.  Measured against the eight-wave kernel on
// the 32 x 32 x 64 form (mx_gemm_tile8.hpp), both in turn: 4096 x 28672 x 8192 E3M2 x E2M1 580 -> 540 us (578 -> 517 and 591 -> 554 on other
// boxes), 2056 to 2075 clocks a step at 1.86 to 1.94 GHz where it was 2210 at 1.74; 16384 x 2048 x 8192 E3M2 178 -> 162 us.  L1 accesses a step of an
// E3M2 pair 1520 -> 1050, cycles of LDS bank conflicts 612 -> 270.  What is left: without the LDS writes a step takes 1640 clocks, without loads and
// writes 1640, matrix instructions alone 1400: with one wave per SIMD an LDS write holds up the instructions behind it.
//
// The scales.  A row's bytes of eight steps are one 32-byte direct load; the rows with (r & 32) == 0 begin such a group at even
// trips of the loop, the others at odd ones, so that each trip requests half the rows' next groups and 16 KB suffice.  A lane
// reads the 16 bytes of a trip's four steps of its row and keeps the byte of block q of each in one register, from which the
// instruction selects the step's.
#pragma once
#include "mx_gemm_tile16.hpp"

#include <type_traits>

namespace mx {
namespace narrow {

// Operand fragment of the instruction: 32 elements of one row, as many registers as they fill
template <int W> struct Frag16 { typedef int type __attribute__((ext_vector_type(W))); };

// One instruction, accumulator updated in place (see mfma16); byte S of both scale registers
template <int H1, int H2, int S, typename V1, typename V2>
__device__ __forceinline__ void mfma16s(v4f_t &acc, const V1 &op1, const V2 &op2, uint32_t s1, uint32_t s2)
{
#ifdef __HIP_DEVICE_COMPILE__        // (a template's assembly is checked against the host's registers, too)
#define MX_ASM(SEL) asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 " SEL " cbsz:%5 blgp:%6" \
                                 : "+a"(acc) : "v"(op1), "v"(op2), "v"(s1), "v"(s2), "n"(H1), "n"(H2))
    if constexpr (S == 0) MX_ASM("op_sel_hi:[0,0,0]");
    else if constexpr (S == 1) MX_ASM("op_sel:[1,1,0] op_sel_hi:[0,0,0]");
    else if constexpr (S == 2) MX_ASM("op_sel_hi:[1,1,0]");
    else MX_ASM("op_sel:[1,1,0] op_sel_hi:[1,1,0]");
#undef MX_ASM
#endif
}

// How an operand tile of 256 rows lies in LDS, where a lane (i, q) finds its fragment of row block 0, and how a line (128 bytes
// of a row: NLINE of them in four K steps) arrives: 16-byte piece c of a line belongs to the first of the line's two steps or (second) the one behind it
template <int W> struct Tile16;
template <> struct Tile16<6> {
    static constexpr int ROW = 96, NP = 3, NLINE = 3, ODD = 16;       // ODD: what flips in the address between 8-row groups
    // chunk c of row r in slot c ^ ((r >> 3) & 1)
    static __device__ __forceinline__ int ofs(int r, int q, int k)
    {
        const int t = 24 * q + 8 * k;
        return r * 96 + (((t >> 4) ^ ((r >> 3) & 1)) << 4) + (t & 8);
    }
    static __device__ __forceinline__ bool second(int l, int c) { return 8 * l + c >= 6 * (l + 1); }
    static __device__ __forceinline__ int put(int r, int l, int c) { return r * 96 + (((8 * l + c) % 6 ^ ((r >> 3) & 1)) << 4); }
};
template <> struct Tile16<4> {
    static constexpr int ROW = 64, NP = 1, NLINE = 2, ODD = 32;
    // chunk c of row r in slot c ^ (-(r >> 2) & 3)
    static __device__ __forceinline__ int ofs(int r, int q, int) { return r * 64 + ((q ^ ((-(r >> 2)) & 3)) << 4); }
    static __device__ __forceinline__ bool second(int, int c) { return c >= 4; }
    static __device__ __forceinline__ int put(int r, int, int c) { return r * 64 + (((c & 3) ^ ((-(r >> 2)) & 3)) << 4); }
};

// A wave-uniform part of an address, kept in a scalar register: the sum with the lane's part is formed where it is used (the
// compiler would rather keep a vector register for every sum of the lane's part with a constant)
__device__ __forceinline__ int uniform(int v)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(v));
#endif
    return v;
}

template <int FA, int FB, int CDT, bool PROBE = false>
__global__ __launch_bounds__(256, 1) void gemm_tile16_kernel(int64_t M, int64_t N, int64_t K,
                                                               const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                                               const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                               void *__restrict__ C, int64_t ldc, int tiles_m, int tiles_n, Raster rast,
                                                               unsigned long long *__restrict__ probe)
{
    unsigned long long probe_c0 = 0, probe_r0 = 0;
    if constexpr (PROBE) { probe_c0 = __builtin_readcyclecounter(); probe_r0 = __builtin_amdgcn_s_memrealtime(); }
    constexpr int WA = Fmt<FA>::bits, WB = Fmt<FB>::bits;
    typedef Tile16<WA> TA;
    typedef Tile16<WB> TB;
    typedef typename Frag16<WA>::type fragA;
    typedef typename Frag16<WB>::type fragB;
    constexpr int A_BYTES = TM * TA::ROW, B_BYTES = TN * TB::ROW, STAGE_BYTES = A_BYTES + B_BYTES;
    constexpr int SC_BYTES = (TM + TN) * 32;             // scale bytes of eight K steps per row
    static_assert(3 * STAGE_BYTES + SC_BYTES <= 160 * 1024, "LDS of a compute unit");
    __shared__ __attribute__((aligned(16))) uint8_t lds[SC_BYTES + 3 * STAGE_BYTES];        // scale bytes, then three stages of {A tile, B tile}
    constexpr int HA = hw_fmt(FA), HB = hw_fmt(FB);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int i = lane & 15, q = lane >> 4;

    int tm, tn;
    if (!raster_tile(rast, (int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * TM, n0 = (int64_t)tn * TN;
    const int64_t nkb = K / BLOCK;
    const int H = (int)(K / (4 * TK));            // trips of the loop: four K steps each

    // ---- staging: wave w brings rows 64w .. 64w+63 of a tile, eight rows a load, one line of each
    const int64_t a_row = K * WA / 8, b_row = K * WB / 8;
    const int r8 = 2 * (lane >> 4) + ((lane >> 2) & 1), c8 = ((lane >> 3) & 1) * 4 + (lane & 3);   // row of the eight, piece of the line
    const uint8_t *gA = Ae + (m0 + wave * 64) * a_row, *gB = Be + (n0 + wave * 64) * b_row;
    const uint32_t va = (uint32_t)(r8 * a_row + c8 * 16), vb = (uint32_t)(r8 * b_row + c8 * 16);
    u32x4_t stA[8], stB[8];
    // byte of the row where line l of trip p begins (trips behind the last: the last again)
    auto line_a = [&](int p, int l) __attribute__((always_inline)) { return (p < H ? p : H - 1) * (64 * WA) + 128 * l; };
    auto line_b = [&](int p, int l) __attribute__((always_inline)) { return (p < H ? p : H - 1) * (64 * WB) + 128 * l; };
    auto load_a = [&](int k, uint32_t v) __attribute__((always_inline)) { return *reinterpret_cast<const u32x4_t *>(gA + k * 8 * a_row + v); };
    auto load_b = [&](int k, uint32_t v) __attribute__((always_inline)) { return *reinterpret_cast<const u32x4_t *>(gB + k * 8 * b_row + v); };
    // where the lane's piece of line l goes: stage `s1`, or the following one, s2.  (The lane's part of an address is made opaque here
    // and below: the compiler would keep a register for every sum of it with a constant.)
    int pla[TA::NLINE], plb[TB::NLINE];
#pragma unroll
    for (int l = 0; l < TA::NLINE; l++) { pla[l] = TA::put(r8, l, c8); asm("" : "+v"(pla[l])); }
#pragma unroll
    for (int l = 0; l < TB::NLINE; l++) { if (WA == WB) plb[l] = pla[l < TA::NLINE ? l : 0]; else { plb[l] = TB::put(r8, l, c8); asm("" : "+v"(plb[l])); } }
    uint32_t later = 0;                   // bit l: the lane's piece of line l of A belongs to the second of its steps; bit 4 + l: of B
#pragma unroll
    for (int l = 0; l < TA::NLINE; l++) later |= TA::second(l, c8) ? 1u << l : 0u;
#pragma unroll
    for (int l = 0; l < TB::NLINE; l++) later |= TB::second(l, c8) ? 16u << l : 0u;
    asm("" : "+v"(later));
    auto put_a = [&](int l, int s1, int s2) __attribute__((always_inline)) {
        return pla[l] + (__builtin_amdgcn_sbfe((int)later, l, 1) & uniform(s2 - s1)) + uniform(wave * (64 * TA::ROW) + s1);
    };
    auto put_b = [&](int l, int s1, int s2) __attribute__((always_inline)) {
        return plb[l] + (__builtin_amdgcn_sbfe((int)later, 4 + l, 1) & uniform(s2 - s1)) + uniform(A_BYTES + wave * (64 * TB::ROW) + s1);
    };
    auto write_a = [&](int k, int v, const u32x4_t &d) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4_t *>(lds + (k & 1 ? v ^ TA::ODD : v) + k * 8 * TA::ROW) = d;
    };
    auto write_b = [&](int k, int v, const u32x4_t &d) __attribute__((always_inline)) {
        *reinterpret_cast<u32x4_t *>(lds + (k & 1 ? v ^ TB::ODD : v) + k * 8 * TB::ROW) = d;
    };
    typedef __attribute__((address_space(3))) void lds_ptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t *)lds);
    // ---- scale bytes
    const uint8_t *sA = As + (m0 + wave * 64) * nkb, *sB = Bs + (n0 + wave * 64) * nkb;
    const uint32_t vs = (uint32_t)((lane & 31) * nkb);
    const int shalf = lane >> 5;
    // rows 32 set .. + 31 of the wave's 64 rows: trips b and b + 1 (clamped to the trips there are)
    auto stage_scales = [&](int set, int b) __attribute__((always_inline)) {
        int u = b + shalf;
        u = u < 0 ? 0 : u < H ? u : H - 1;
        const uint32_t vo = vs + 16 * u;
        const uint8_t *pa = sA + set * 32 * nkb, *pb = sB + set * 32 * nkb;
        const uint32_t l0 = lds0 + wave * 2048 + set * 1024;
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(vo), "s"(pa), "s"(l0) : "m0");
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(vo), "s"(pb), "s"(l0 + 8192) : "m0");
    };

    v4f_t acc[8][8];
#pragma unroll
    for (int x = 0; x < 8; x++)
#pragma unroll
        for (int y = 0; y < 8; y++) acc[x][y] = v4f_t{0.f, 0.f, 0.f, 0.f};

    // ---- operand reads
    int oa[TA::NP], ob[TB::NP];           // the lane's part (128 rows further: the same swizzle)
#pragma unroll
    for (int k = 0; k < TA::NP; k++) { oa[k] = TA::ofs(i, q, k); asm("" : "+v"(oa[k])); }
#pragma unroll
    for (int k = 0; k < TB::NP; k++) { if (WA == WB) ob[k] = oa[k < TA::NP ? k : 0]; else { ob[k] = TB::ofs(i, q, k); asm("" : "+v"(ob[k])); } }
    const int wofs_a = wm * 128 * TA::ROW, wofs_b = A_BYTES + wn * 128 * TB::ROW;
    // piece k of the fragment of 16-row block xb of the stage last aimed at
    int ad_a[TA::NP], ad_b[TB::NP];
    auto aim_a = [&](int st) __attribute__((always_inline)) {
        const int u = uniform(st + wofs_a);
#pragma unroll
        for (int k = 0; k < TA::NP; k++) ad_a[k] = oa[k] + u;
    };
    auto aim_b = [&](int st) __attribute__((always_inline)) {
        const int u = uniform(st + wofs_b);
#pragma unroll
        for (int k = 0; k < TB::NP; k++) ad_b[k] = ob[k] + u;
    };
    auto read_a = [&](fragA &f, int xb, int k) __attribute__((always_inline)) {
        const uint8_t *p = lds + ad_a[k] + xb * (16 * TA::ROW);
        if constexpr (WA == 6) { const uint2 d = *reinterpret_cast<const uint2 *>(p); f[2 * k] = (int)d.x; f[2 * k + 1] = (int)d.y; }
        else { const uint4 d = *reinterpret_cast<const uint4 *>(p); f[0] = (int)d.x; f[1] = (int)d.y; f[2] = (int)d.z; f[3] = (int)d.w; }
    };
    auto read_b = [&](fragB &f, int xb, int k) __attribute__((always_inline)) {
        const uint8_t *p = lds + ad_b[k] + xb * (16 * TB::ROW);
        if constexpr (WB == 6) { const uint2 d = *reinterpret_cast<const uint2 *>(p); f[2 * k] = (int)d.x; f[2 * k + 1] = (int)d.y; }
        else { const uint4 d = *reinterpret_cast<const uint4 *>(p); f[0] = (int)d.x; f[1] = (int)d.y; f[2] = (int)d.z; f[3] = (int)d.w; }
    };
    fragA aL[4], aH[4];
    fragB bL[4], bH[4];
    uint32_t sa[8], sb[8], na[4], nb[4];  // byte h: scale of row / column i, block q, step h of the trip; na / nb: next trip, blocks 4-7
    u32x4_t raw[2];
    // scale reads of trip p: the 16 bytes of row i of blocks x0 and x0 + 1
    int rs = i * 16;
    asm("" : "+v"(rs));
    auto read_raw = [&](int p, bool isb, int x0) __attribute__((always_inline)) {
        p = p < H ? p : H - 1;
        const int set = (x0 >> 1) & 1, half = (p & 1) ^ set;          // set 0's pairs of trips start at even ones, set 1's at odd ones
#pragma unroll
        for (int x = 0; x < 2; x++)
            raw[x] = *reinterpret_cast<const u32x4_t *>(lds + (rs + uniform(half * 512 + (isb ? wn * 4096 : wm * 4096))) + (isb ? 8192 : 0) + (x0 >> 2) * 2048 + set * 1024 + x * 256);
    };
    const uint32_t sel_lo = (uint32_t)(q | (4 + q) << 8 | 0x0c0c0000), sel_hi = (uint32_t)(q << 16 | (4 + q) << 24 | 0x0c0c);
    auto gather = [&](const u32x4_t &r) __attribute__((always_inline)) {
        return __builtin_amdgcn_perm(r[1], r[0], sel_lo) | __builtin_amdgcn_perm(r[3], r[2], sel_hi);
    };
    auto take_raw = [&](uint32_t *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 2; x++) dst[x] = gather(raw[x]);
    };
#define MX_FENCE() __builtin_amdgcn_sched_barrier(0)

    // ---- prologue: the lines of steps 0 and 1 that the first step cannot do without (of B only the first: its second is written
    // during that step, as everywhere), then those that are written next
    {
        u32x4_t a0[8], b0[8], a1[8];
        stage_scales(0, 0);
        stage_scales(1, -1);
#pragma unroll
        for (int k = 0; k < 8; k++) { a0[k] = load_a(k, va); b0[k] = load_b(k, vb); }
        if (TA::NLINE == 3) {
#pragma unroll
            for (int k = 0; k < 8; k++) a1[k] = load_a(k, va + 128);
        }
#pragma unroll
        for (int k = 0; k < 8; k++) stB[k] = load_b(k, vb + 128);
#pragma unroll
        for (int k = 0; k < 8; k++) stA[k] = load_a(k, va + 128 * (TA::NLINE - 1));
        const int s0 = SC_BYTES, s1 = SC_BYTES + STAGE_BYTES, s2 = SC_BYTES + 2 * STAGE_BYTES;
        const int pa0 = put_a(0, s0, s1), pb0 = put_b(0, s0, s1), pa1 = put_a(1, s1, s2);
#pragma unroll
        for (int k = 0; k < 8; k++) { write_a(k, pa0, a0[k]); write_b(k, pb0, b0[k]); }
        if (TA::NLINE == 3) {
#pragma unroll
            for (int k = 0; k < 8; k++) write_a(k, pa1, a1[k]);
        }
    }
    __syncthreads();        // (the scale bytes were requested before the lines that have been waited for)
    int cur = SC_BYTES, nxt = SC_BYTES + STAGE_BYTES, prv = SC_BYTES + 2 * STAGE_BYTES;   // stages of steps t, t + 1 and t + 2
    aim_a(cur); aim_b(cur);
#pragma unroll
    for (int x = 0; x < 4; x++)
#pragma unroll
        for (int k = 0; k < TA::NP; k++) read_a(aL[x], x, k);
#pragma unroll
    for (int x = 0; x < 4; x++)
#pragma unroll
        for (int k = 0; k < TB::NP; k++) read_b(bL[x], x, k);
#pragma unroll
    for (int x = 0; x < 8; x += 2) {
        read_raw(0, false, x); take_raw(sa + x);
        read_raw(0, true, x); take_raw(sb + x);
    }

    auto quad = [&](auto hc, auto &AS, auto &BS, auto xc, auto yc, auto &&slot) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value, X0 = decltype(xc)::value, Y0 = decltype(yc)::value;
#pragma unroll
        for (int m = 0; m < 16; m++) {
            slot(m);
            const int x = m & 3, y = m >> 2;
            mfma16s<HB, HA, h>(acc[X0 + x][Y0 + y], BS[y], AS[x], sb[Y0 + y], sa[X0 + x]);
            MX_FENCE();
        }
    };
    auto quadT = [&](auto hc, auto &AS, auto &BS, auto xc, auto yc, auto &&slot) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value, X0 = decltype(xc)::value, Y0 = decltype(yc)::value;
#pragma unroll
        for (int m = 0; m < 16; m++) {
            slot(m);
            const int x = m >> 2, y = m & 3;
            mfma16s<HB, HA, h>(acc[X0 + x][Y0 + y], BS[y], AS[x], sb[Y0 + y], sa[X0 + x]);
            MX_FENCE();
        }
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 4> c4{};
    // Window h (Q3 and Q4 of step h, Q1 and Q2 of the next): which line of which operand is written (-1: none).  Its registers
    // take the following line at once.
    auto line_of = [](int w, int h) __attribute__((always_inline)) { return w == 6 ? (h == 0 ? 2 : h == 2 ? 0 : h == 3 ? 1 : -1) : (h == 0 ? 1 : h == 2 ? 0 : -1); };
    auto k_step = [&](auto hc, const int p) __attribute__((always_inline)) {
        constexpr int h = decltype(hc)::value, hp = (h + 3) & 3;
        MX_FENCE();
        auto &B1 = *((h & 1) ? &bH : &bL);        // used in Q1 and Q4
        auto &B2 = *((h & 1) ? &bL : &bH);        // refilled in Q1, used in Q2 and Q3
        constexpr int Y1 = (h & 1) ? 4 : 0, Y2 = 4 - Y1;
        constexpr std::integral_constant<int, Y1> y1{};
        constexpr std::integral_constant<int, Y2> y2{};
        constexpr int RB = 4 * TB::NP, RA = 4 * TA::NP;
        // reads r of the first half: the other B half, then aH
        auto rd1 = [&](int r) __attribute__((always_inline)) {
            if (r < RB) read_b(B2[r / TB::NP], Y2 + r / TB::NP, r % TB::NP);
            else if (r - RB < RA) read_a(aH[(r - RB) / TA::NP], 4 + (r - RB) / TA::NP, (r - RB) % TA::NP);
        };
        // B's share of the previous step's window, A's of this one's
        const int lb = line_of(WB, hp), la = line_of(WA, h);
        const int pb = lb == TB::NLINE - 1 ? (h == 1 ? p + 1 : p) : h == 0 ? p : p + 1;        // trip of the line that follows line lb
        const int pa = p + 1;                                                                   // (windows 0, 2, 3: always the next trip's)
        aim_a(cur); aim_b(cur);
        int wb = 0, wa = 0;
        uint32_t xb = 0, xa = 0;
        if (lb >= 0) { wb = put_b(lb, nxt, prv); xb = vb + uniform(line_b(pb, lb == TB::NLINE - 1 ? 0 : lb + 1)); }
        auto move_b = [&](int k) __attribute__((always_inline)) { if (lb >= 0) { write_b(k, wb, stB[k]); } };
        auto next_b = [&](int k) __attribute__((always_inline)) { if (lb >= 0) { stB[k] = load_b(k, xb); } };
        quad(hc, aL, B1, c0, y1, [&](int m) __attribute__((always_inline)) {
            if (h == 3 && m == 12) take_raw(nb + 2);
            rd1(m);
            if ((m & 3) == 1) move_b(m >> 2);
            if ((m & 3) == 2) next_b(m >> 2);
        });
        quad(hc, aL, B2, c0, y2, [&](int m) __attribute__((always_inline)) {
            if (h == 3 && m == 12) read_raw(p + 1, false, 0);
            if (m < 8) rd1(16 + m);
            if (m < 8 && (m & 1) == 0) move_b(4 + m / 2);
            if (m < 8 && (m & 1) == 1) next_b(4 + m / 2);
        });
        // stage t+1 is in LDS and every wave has its last read of stage t behind it
        if (h == 2) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");        // the scale bytes requested two steps ago, before 16 loads
        __syncthreads();
        MX_FENCE();
        aim_a(nxt); aim_b(nxt);
        if (la >= 0) { wa = put_a(la, prv, cur); xa = va + uniform(line_a(pa, la == TA::NLINE - 1 ? 0 : la + 1)); }
        auto move_a = [&](int k) __attribute__((always_inline)) { if (la >= 0) { write_a(k, wa, stA[k]); } };
        auto next_a = [&](int k) __attribute__((always_inline)) { if (la >= 0) { stA[k] = load_a(k, xa); } };
        quadT(hc, aH, B2, c4, y2, [&](int m) __attribute__((always_inline)) {
            if (h == 0 && m == 0) stage_scales((p & 1) ^ 1, p + 1);
            if (h == 2 && m == 4) read_raw(p + 1, false, 4);
            if (h == 2 && m == 12) { take_raw(na); read_raw(p + 1, false, 6); }
            if (h == 3 && m == 4) { take_raw(sa); read_raw(p + 1, false, 2); }
            if (h == 3 && m == 12) { take_raw(sa + 2); read_raw(p + 1, true, 0); }
            if (m < RA) read_a(aL[m / TA::NP], m / TA::NP, m % TA::NP);
            if ((m & 3) == 1) move_a(m >> 2);
            if ((m & 3) == 2) next_a(m >> 2);
        });
        quadT(hc, aH, B1, c4, y1, [&](int m) __attribute__((always_inline)) {
            if (h == 2 && m == 4) { take_raw(na + 2); read_raw(p + 1, true, 4); }
            if (h == 2 && m == 12) { take_raw(nb); read_raw(p + 1, true, 6); }
            if (h == 3 && m == 4) { take_raw(sb); read_raw(p + 1, true, 2); }
            if (h == 3 && m == 12) take_raw(sb + 2);
            if (m < RB) read_b(B2[m / TB::NP], Y2 + m / TB::NP, m % TB::NP);
            if ((m & 3) == 1) move_a(4 + (m >> 2));
            if ((m & 3) == 2) next_a(4 + (m >> 2));
        });
        if (h == 3) {
#pragma unroll
            for (int x = 0; x < 4; x++) { sa[4 + x] = na[x]; sb[4 + x] = nb[x]; }
            MX_FENCE();
            asm volatile("s_nop 1");          // vector write of a scale register -> matrix instruction
        }
        const int free = cur;
        cur = nxt; nxt = prv; prv = free;
        MX_FENCE();
    };
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, 2> c2{};
    constexpr std::integral_constant<int, 3> c3{};
    for (int p = 0; p < H; p++) {
        k_step(c0, p);
        k_step(c1, p);
        k_step(c2, p);
        k_step(c3, p);
    }
#undef MX_FENCE
    acc_settle(acc);
    if constexpr (PROBE) {
        if (threadIdx.x == 0) {
            probe[2 * blockIdx.x] = __builtin_readcyclecounter() - probe_c0;
            probe[2 * blockIdx.x + 1] = __builtin_amdgcn_s_memrealtime() - probe_r0;
        }
    }
    store_tile16<CDT>(acc, C, ldc, m0 + wm * 128, n0 + wn * 128, i, q);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // scale bytes requested behind the last trip must have landed before the LDS is given up
}

}  // namespace narrow

template <int FA, int FB, int CDT>
static hipError_t launch_t16n(const TileArgs &a)
{
    auto kern = narrow::gemm_tile16_kernel<FA, FB, CDT>;
    const int tiles_m = (int)(a.M / TM), tiles_n = (int)(a.N / TN);
    const Raster rast = choose_raster(tiles_m, tiles_n, Fmt<FA>::bits, Fmt<FB>::bits);
    hipLaunchKernelGGL(kern, dim3(raster_grid(rast, tiles_m, tiles_n)), dim3(256), 0, a.st, a.M, a.N, a.K, a.Ae, a.As, a.Be, a.Bs, a.C, a.ldc,
                       tiles_m, tiles_n, rast, static_cast<unsigned long long *>(nullptr));
    return hipGetLastError();
}

template <int FA, int FB>
static hipError_t launch_pair16n(const TileArgs &a)
{
    return a.c_dt == DT_F32 ? launch_t16n<FA, FB, DT_F32>(a) : launch_t16n<FA, FB, DT_BF16>(a);
}

template <int FA>
static hipError_t launch_a16n(const TileArgs &a, int fmtB)
{
    if (fmtB == FP6_E3M2) return launch_pair16n<FA, FP6_E3M2>(a);
    if (fmtB == FP6_E2M3) return launch_pair16n<FA, FP6_E2M3>(a);
    if constexpr (Fmt<FA>::bits == 6) {
        if (fmtB == FP4_E2M1) return launch_pair16n<FA, FP4_E2M1>(a);
    }
    return hipErrorNotSupported;
}

}  // namespace mx
