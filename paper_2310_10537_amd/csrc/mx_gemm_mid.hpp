// LDS-tiled MX GEMM for the problems that 256 x 256 tiles do not fit (Section 4.1 of arXiv 2310.10537): any
// M and N, any K of whole blocks.
//
// Work-group: four waves in a 2 x 2 arrangement, output tile BM x BN with BM = 64 * MB, BN = 64 * NB, K step 128;
// a wave owns MB x NB tiles of the 32x32x64 block-scaled matrix instruction.  Operands reach LDS by direct loads
// into NSTAGE buffers, laid out exactly as in mx_gemm_tile.hpp (same swizzles, same operand reads); rows beyond M
// and columns beyond N read the last valid one instead and are not stored.  Scale bytes travel the same way,
// 16 bytes per row -- four K steps -- at a time.  A last K step of fewer than 128 elements goes through registers, zero-filled.
//
// An entry's products are chained in increasing K, 64 at a time, as in the direct and the 256 x 256 kernels: the same bits.
#pragma once

#include "mx_gemm_tile.hpp"

namespace mx {

typedef uint32_t u32x4_unaligned __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_al8 __attribute__((ext_vector_type(2)));

// 16 scale bytes of one row, blocks kb .. kb + 15, as four dwords.
// Blocks at and beyond nkb come back as 0 (their elements are zero as well, so the value does not matter).
__device__ __forceinline__ void load_scale_group(const uint8_t *row, int64_t kb, int64_t nkb, uint32_t (&d)[4])
{
    if (kb + 16 <= nkb) {
        const u32x4_unaligned v = *reinterpret_cast<const u32x4_unaligned *>(row + kb);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    } else if (nkb >= 16) {                                   // the row's last 16 bytes, moved down by whole bytes (wave-uniform)
        const u32x4_unaligned v = *reinterpret_cast<const u32x4_unaligned *>(row + nkb - 16);
        const int sh = (int)(kb + 16 - nkb);                  // 1 .. 15
        const uint64_t lo = ((uint64_t)v.y << 32) | v.x, hi = ((uint64_t)v.w << 32) | v.z;
        uint64_t rl, rh;
        if (sh >= 8) { rl = hi >> (8 * (sh - 8)); rh = 0; }
        else { rl = (lo >> (8 * sh)) | (hi << (64 - 8 * sh)); rh = hi >> (8 * sh); }
        d[0] = (uint32_t)rl; d[1] = (uint32_t)(rl >> 32); d[2] = (uint32_t)rh; d[3] = (uint32_t)(rh >> 32);
    } else {                                                  // fewer than 512 elements in all
#pragma unroll
        for (int q = 0; q < 4; q++) {
            d[q] = 0;
#pragma unroll
            for (int b = 0; b < 4; b++)
                if (kb + 4 * q + b < nkb) d[q] |= (uint32_t)row[kb + 4 * q + b] << (8 * b);
        }
    }
}

template <int FA, int FB, int MB, int NB, int NSTAGE>
__global__ __launch_bounds__(256, 2) void gemm_mid_kernel(int M, int N, int64_t K, const uint8_t *__restrict__ Ae,
                                                          const uint8_t *__restrict__ As, const uint8_t *__restrict__ Be,
                                                          const uint8_t *__restrict__ Bs, void *__restrict__ C, int c_dt, int64_t ldc,
                                                          int tiles_m, int tiles_n, Raster rast)
{
    constexpr int WA = Fmt<FA>::bits, WB = Fmt<FB>::bits;
    constexpr int HA = hw_fmt(FA), HB = hw_fmt(FB);   // must reach the builtin as literal constants
    // FA = FB = INT8: bf16 operands without scales, K counts the bytes of a row (64 elements a step), and the two 16-byte chunks of a
    // lane are the operands of two 32 x 32 x 16 bf16 instructions; everything else is the same, but for the sums.  The bf16 instruction
    // rounds the running sum several times, so its chains are kept short and their results added to sums of their own:
    //  - LEVELS = 2 (128 x 128 tiles): chains of `chain` steps, one sum of them;
    //  - LEVELS = 3 (tiles of half the size: three sets of accumulators fill the registers of two waves per SIMD otherwise): both halves of
    //    a step -- an MXINT8 block each, whose sum is exact -- apart, added to each other and to the sum of `each` steps, about the root of
    //    their number, that one to the sum of all.
    // Error (2-norm, scales spread over 16 octaves, K = 4096): one chain 3.4e-7, LEVELS = 2 1.3e-7, LEVELS = 3 0.8e-7.
    constexpr bool BF = FA == INT8 && FB == INT8;
    constexpr int LEVELS = !BF ? 1 : MB * NB > 2 ? 2 : 3;
    constexpr int BM = 64 * MB, BN = 64 * NB;
    // wave-wide direct loads (1 KB) per wave and operand; a 6-bit tile of 64 rows (6 KB) is padded to 8 KB
    constexpr int NJA = (BM * TileFmt<WA>::ROW + 4095) / 4096, NJB = (BN * TileFmt<WB>::ROW + 4095) / 4096, NJ = NJA + NJB;
    constexpr int A_BYTES = NJA * 4096, STAGE_BYTES = NJ * 4096;
    constexpr int SG_BYTES = (MB + NB) * 1024;               // one group of scale bytes; two of them behind the stages
    __shared__ __attribute__((aligned(16))) uint8_t lds[NSTAGE * STAGE_BYTES + 2 * SG_BYTES];
    static_assert(sizeof(lds) <= 160 * 1024, "LDS of a compute unit");
    uint8_t *const scl = lds + NSTAGE * STAGE_BYTES;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1, i = lane & 31, g = lane >> 5;

    int tm, tn;
    if (!raster_tile(rast, (int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * BM, n0 = tn * BN;
    const int64_t nkb = K / BLOCK;
    const int T = (int)(K / TK);                              // whole K steps
    const int tail = (int)(K - (int64_t)T * TK);              // 0, 32, 64 or 96 more elements
    const uint32_t a_row = (uint32_t)(K * WA / 8), b_row = (uint32_t)(K * WB / 8);

    // ---- staging map: slot n = (4j + wave) * 64 + lane of the tile -> (row, 16-byte piece) the layout keeps there
    auto slot_row = [](int w, int n) { return w == 8 ? n >> 3 : w == 4 ? n >> 2 : n / 6; };
    auto slot_piece = [](int w, int n, int r) {
        return w == 8 ? (n & 7) ^ ((r >> 1) & 7) : w == 4 ? (n & 3) ^ ((r >> 2) & 3) : (n - 6 * r) ^ ((r >> 3) & 1);
    };
    uint32_t oa[NJA], ob[NJB];                                // byte offsets from the tile's first row
    int pa[NJA], pb[NJB];                                     // pieces (the last, partial step looks at them)
#pragma unroll
    for (int j = 0; j < NJA; j++) {
        const int n = (4 * j + wave) * 64 + lane, r = slot_row(WA, n);
        pa[j] = slot_piece(WA, n, r);
        oa[j] = (uint32_t)(m0 + r < M ? r : M - 1 - m0) * a_row + pa[j] * 16;
    }
#pragma unroll
    for (int j = 0; j < NJB; j++) {
        const int n = (4 * j + wave) * 64 + lane, r = slot_row(WB, n);
        pb[j] = slot_piece(WB, n, r);
        ob[j] = (uint32_t)(n0 + r < N ? r : N - 1 - n0) * b_row + pb[j] * 16;
    }
    const uint8_t *gA = Ae + (int64_t)m0 * a_row, *gB = Be + (int64_t)n0 * b_row;
    typedef __attribute__((address_space(3))) void lds_ptr_t;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t *)lds) + wave * 1024;
    const uint32_t scl0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t *)scl);
    // direct load number k (A's, then B's) of K step t into the buffer at byte offset dst
    auto stage_one = [&](int k, int t, int dst) {
        t = t < T ? t : T - 1;                                // past the end: the last step again, never used
        const uint32_t l = lds0 + dst + k * 4096;
        if (k < NJA) {
            const uint8_t *p = gA + (int64_t)t * (TK * WA / 8);
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(oa[k < NJA ? k : 0]), "s"(p), "s"(l) : "m0", "memory");
        } else {
            const uint8_t *p = gB + (int64_t)t * (TK * WB / 8);
            asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(ob[k < NJA ? 0 : k - NJA]), "s"(p), "s"(l) : "m0", "memory");
        }
    };

    // ---- scale bytes, 16 per row (four K steps) at a time: wave w brings the rows 64 w .. 64 w + 63 of {A tile, B tile}.
    // Direct loads where a row's groups are dword-aligned and 16 bytes long; else through registers, zero-filled.
    // The partial last group is loaded as the row's last 16 bytes and its steps sit further back in the slot.
    const bool direct_scales = nkb % 4 == 0 && nkb >= 16;
    const int steps = T + (tail > 0), n_groups = (steps + 3) / 4;
    const int seg = wave < MB + NB ? wave : MB + NB - 1;      // (a spare wave repeats the last segment)
    const uint8_t *srow;
    if (seg < MB) srow = As + (int64_t)(m0 + seg * 64 + lane < M ? m0 + seg * 64 + lane : M - 1) * nkb;
    else srow = Bs + (int64_t)(n0 + (seg - MB) * 64 + lane < N ? n0 + (seg - MB) * 64 + lane : N - 1) * nkb;
    auto stage_scales = [&](int G) {
        if constexpr (BF) return;
        if (direct_scales) {
            const uint32_t l = scl0 + (G & 1) * SG_BYTES + seg * 1024;
            const uint8_t *p = srow + (4 * G + 4 <= steps ? 16 * G : 4 * steps - 16);
            asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(p), "s"(l) : "m0", "memory");
        } else {
            uint32_t d[4];
            load_scale_group(srow, 16 * (int64_t)G, nkb, d);
            *reinterpret_cast<uint4 *>(scl + (G & 1) * SG_BYTES + seg * 1024 + lane * 16) = make_uint4(d[0], d[1], d[2], d[3]);
        }
    };
    uint32_t sa[MB] = {}, sb[NB] = {};
    // scale dwords of step t; lanes 32 .. 63 shift theirs by a byte: one selector then addresses block 2 sub + g
    auto read_scales = [&](int t) {
        if constexpr (BF) return;
        t = t < steps ? t : steps - 1;
        const int pos = direct_scales && (t | 3) >= steps ? t - steps + 4 : t & 3;
        const uint8_t *s = scl + ((t >> 2) & 1) * SG_BYTES + pos * 4;
#pragma unroll
        for (int x = 0; x < MB; x++) sa[x] = *reinterpret_cast<const uint32_t *>(s + (wm * (BM / 2) + 32 * x + i) * 16) >> (8 * g);
#pragma unroll
        for (int y = 0; y < NB; y++) sb[y] = *reinterpret_cast<const uint32_t *>(s + (BM + wn * (BN / 2) + 32 * y + i) * 16) >> (8 * g);
    };

    const FragOfs<WA> fa = frag_ofs<WA>(wm * (BM / 2) + i, g);
    const FragOfs<WB> fb = frag_ofs<WB>(wn * (BN / 2) + i, g);
    v16f_t acc[MB][NB];
#pragma unroll
    for (int x = 0; x < MB; x++)
#pragma unroll
        for (int y = 0; y < NB; y++)
#pragma unroll
            for (int t = 0; t < 16; t++) acc[x][y][t] = 0.f;
    // LEVELS > 1: acc is the first half step's chain or the running one
    v16f_t acc1[MB][NB], run[MB][NB], sum[MB][NB];            // the second half step's chain; sums of `each` steps; of everything
    const int chain = K < 1024 ? 1 : K < 2048 ? 4 : 8;        // (LEVELS = 2; the shorter K, the fewer roundings to stay below)
    int each = 4;
    while (LEVELS == 3 && each * each * 3 / 2 < T) each *= 2;
    if constexpr (LEVELS > 1) {
#pragma unroll
        for (int x = 0; x < MB; x++)
#pragma unroll
            for (int y = 0; y < NB; y++) { run[x][y] = acc[x][y]; sum[x][y] = acc[x][y]; }
    }

    v8i_t a0[MB], b0[NB], a1[MB], b1[NB];                     // operands of sub-step 0 / 1
    auto read_sub = [&](const uint8_t *buf, int sub, v8i_t (&a)[MB], v8i_t (&b)[NB]) {
#pragma unroll
        for (int x = 0; x < MB; x++) a[x] = read_frag<WA>(buf, fa, sub, x);
#pragma unroll
        for (int y = 0; y < NB; y++) b[y] = read_frag<WB>(buf + A_BYTES, fb, sub, y);
    };
    // B goes first: a lane ends up with groups of four consecutive columns of one row of C
    auto mid_bf16 = [](const v8i_t &b, const v8i_t &a, v16f_t c) __attribute__((always_inline)) {
        typedef __bf16 bf16x8_t_ __attribute__((ext_vector_type(8)));
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t_, __builtin_shufflevector(b, b, 0, 1, 2, 3)),
                                                    __builtin_bit_cast(bf16x8_t_, __builtin_shufflevector(a, a, 0, 1, 2, 3)), c, 0, 0, 0);
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t_, __builtin_shufflevector(b, b, 4, 5, 6, 7)),
                                                       __builtin_bit_cast(bf16x8_t_, __builtin_shufflevector(a, a, 4, 5, 6, 7)), c, 0, 0, 0);
    };
    constexpr v16f_t zero = {};
#define MX_MID_MFMA(SUB, A_, B_, X, Y)                                                                                              \
    do {                                                                                                                            \
        if constexpr (LEVELS == 3 && SUB == 0) acc[X][Y] = mid_bf16(B_[Y], A_[X], zero);                                            \
        else if constexpr (LEVELS == 3) acc1[X][Y] = mid_bf16(B_[Y], A_[X], zero);                                                  \
        else if constexpr (BF) acc[X][Y] = mid_bf16(B_[Y], A_[X], acc[X][Y]);                                                       \
        else acc[X][Y] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(B_[Y], A_[X], acc[X][Y], HB, HA, 2 * SUB, (int)sb[Y], 2 * SUB, (int)sa[X]); \
    } while (0)
    // behind step t (LEVELS > 1)
    auto add_up = [&](int t, bool second) __attribute__((always_inline)) {
        if constexpr (LEVELS == 3) {
#pragma unroll
            for (int x = 0; x < MB; x++)
#pragma unroll
                for (int y = 0; y < NB; y++) run[x][y] += second ? acc[x][y] + acc1[x][y] : acc[x][y];
            if ((t & (each - 1)) == each - 1) {
#pragma unroll
                for (int x = 0; x < MB; x++)
#pragma unroll
                    for (int y = 0; y < NB; y++) { sum[x][y] += run[x][y]; run[x][y] = zero; }
            }
        } else if constexpr (LEVELS == 2) {
            if ((t + 1) % chain == 0) {
#pragma unroll
                for (int x = 0; x < MB; x++)
#pragma unroll
                    for (int y = 0; y < NB; y++) { sum[x][y] += acc[x][y]; acc[x][y] = zero; }
            }
        }
    };

    stage_scales(0);
    if (T > 0) {
        // Pipeline: a step's second half of operands is read beside the matrix instructions of its first half, the
        // next step's first half beside those of its second; the one barrier stands between the two, where every
        // read of the step's buffer has been issued and the next step's must have landed.  Behind it the buffer takes
        // the step NSTAGE further on.
#pragma unroll
        for (int s = 0; s < NSTAGE; s++)
#pragma unroll
            for (int k = 0; k < NJ; k++) stage_one(k, s, s * STAGE_BYTES);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 1) * NJ) : "memory");
        __syncthreads();
        read_scales(0);
        read_sub(lds, 0, a0, b0);
        int buf = 0;                                          // byte offset of step t's buffer
        for (int t = 0; t < T; t++) {
            const int nxt = buf + STAGE_BYTES == NSTAGE * STAGE_BYTES ? 0 : buf + STAGE_BYTES;
            read_sub(lds + buf, 1, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < MB; x++)
#pragma unroll
                for (int y = 0; y < NB; y++) MX_MID_MFMA(0, a0, b0, x, y);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 2) * NJ) : "memory");
            __syncthreads();
            if ((t & 3) == 0 && (t >> 2) + 1 < n_groups) stage_scales((t >> 2) + 1);
            read_sub(lds + nxt, 0, a0, b0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int x = 0; x < MB; x++)
#pragma unroll
                for (int y = 0; y < NB; y++) {
                    constexpr int PER = (NJ + MB * NB - 1) / (MB * NB);   // direct loads per matrix instruction
#pragma unroll
                    for (int k = 0; k < PER; k++)
                        if ((x * NB + y) * PER + k < NJ) stage_one((x * NB + y) * PER + k, t + NSTAGE, buf);
                    MX_MID_MFMA(1, a1, b1, x, y);
                    __builtin_amdgcn_sched_barrier(0);
                }
            read_scales(t + 1);
            add_up(t, true);
            buf = nxt;
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // requests past the end: landed before LDS is reused
    if (tail) {
        __syncthreads();
        // 24 bytes per 6-bit block: a piece may hold 8 valid bytes
        auto piece = [&](const uint8_t *p, int valid) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (valid > 0) { const u32x2_al8 d = *reinterpret_cast<const u32x2_al8 *>(p); v.x = d.x; v.y = d.y; }
            if (valid > 8) { const u32x2_al8 d = *reinterpret_cast<const u32x2_al8 *>(p + 8); v.z = d.x; v.w = d.y; }
            return v;
        };
#pragma unroll
        for (int j = 0; j < NJA; j++)
            *reinterpret_cast<uint4 *>(lds + wave * 1024 + lane * 16 + j * 4096) =
                piece(gA + (int64_t)T * (TK * WA / 8) + oa[j], tail * WA / 8 - pa[j] * 16);
#pragma unroll
        for (int j = 0; j < NJB; j++)
            *reinterpret_cast<uint4 *>(lds + A_BYTES + wave * 1024 + lane * 16 + j * 4096) =
                piece(gB + (int64_t)T * (TK * WB / 8) + ob[j], tail * WB / 8 - pb[j] * 16);
        __syncthreads();
        read_scales(T);
        read_sub(lds, 0, a0, b0);
        read_sub(lds, 1, a1, b1);
#pragma unroll
        for (int x = 0; x < MB; x++)
#pragma unroll
            for (int y = 0; y < NB; y++) {
                MX_MID_MFMA(0, a0, b0, x, y);
                if (tail > 64) MX_MID_MFMA(1, a1, b1, x, y);
            }
        if constexpr (LEVELS == 3) add_up(T, tail > 64);
    }
#undef MX_MID_MFMA
    if constexpr (LEVELS > 1) {
#pragma unroll
        for (int x = 0; x < MB; x++)
#pragma unroll
            for (int y = 0; y < NB; y++) acc[x][y] = sum[x][y] + (LEVELS == 3 ? run[x][y] : acc[x][y]);
    }

    // ---- epilogue: result register t of instruction tile (x, y): row i, column 8 (t / 4) + 4g + t % 4.  bf16: the two
    // half-waves trade groups of four columns, so that each lane stores eight consecutive ones (columns 16 h + 8g ..).
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t_ __attribute__((ext_vector_type(2)));
    auto pack2 = [](float lo, float hi) {
        const f32x2_t v = {lo, hi};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t_));
    };
    const bool wide = c_dt == DT_F32 ? (ldc & 3) == 0 : (ldc & 7) == 0;
#pragma unroll
    for (int x = 0; x < MB; x++) {
        const int r = m0 + wm * (BM / 2) + 32 * x + i;
        if (r >= M) continue;                                 // (both half-waves hold the same rows)
        const int64_t row = (int64_t)r * ldc;
#pragma unroll
        for (int y = 0; y < NB; y++) {
            const int c0 = n0 + wn * (BN / 2) + 32 * y;
            if (c_dt == DT_F32) {
                float *o = reinterpret_cast<float *>(C) + row;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int c = c0 + 8 * q + 4 * g;
                    if (wide && c + 4 <= N)
                        *reinterpret_cast<float4 *>(o + c) = make_float4(acc[x][y][4 * q], acc[x][y][4 * q + 1], acc[x][y][4 * q + 2], acc[x][y][4 * q + 3]);
                    else
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            if (c + e < N) o[c + e] = acc[x][y][4 * q + e];
                }
            } else {
                uint16_t *o = reinterpret_cast<uint16_t *>(C) + row;
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const v16f_t &v = acc[x][y];
                    const auto lo = __builtin_amdgcn_permlane32_swap(pack2(v[8 * h], v[8 * h + 1]), pack2(v[8 * h + 4], v[8 * h + 5]), false, false);
                    const auto hi = __builtin_amdgcn_permlane32_swap(pack2(v[8 * h + 2], v[8 * h + 3]), pack2(v[8 * h + 6], v[8 * h + 7]), false, false);
                    const int c = c0 + 16 * h + 8 * g;
                    const uint32_t d[4] = {lo[0], hi[0], lo[1], hi[1]};
                    if (wide && c + 8 <= N) *reinterpret_cast<uint4 *>(o + c) = make_uint4(d[0], d[1], d[2], d[3]);
                    else
#pragma unroll
                        for (int e = 0; e < 8; e++)
                            if (c + e < N) o[c + e] = (uint16_t)(d[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
    }
}

template <int FA, int FB, int MB, int NB, int NSTAGE>
static hipError_t launch_mid_t(const TileArgs &a)
{
    const int tiles_m = (int)((a.M + 64 * MB - 1) / (64 * MB)), tiles_n = (int)((a.N + 64 * NB - 1) / (64 * NB));
    const Raster rast = choose_raster(tiles_m, tiles_n, Fmt<FA>::bits, Fmt<FB>::bits);
    hipLaunchKernelGGL((gemm_mid_kernel<FA, FB, MB, NB, NSTAGE>), dim3(raster_grid(rast, tiles_m, tiles_n)), dim3(256), 0, a.st, (int)a.M,
                       (int)a.N, a.K, a.Ae, a.As, a.Be, a.Bs, a.C, a.c_dt, a.ldc, tiles_m, tiles_n, rast);
    return hipGetLastError();
}

// The tile: the smallest of 64 x 64, 64 x 128 and 128 x 128 whose tiles all run at once, one per compute unit -- a smaller one takes a
// second round and re-reads the operands more often, a larger one leaves compute units idle; 128 x 128 where none does.  E4M3 pairs, 64 x 64 / 64 x 128 /
// 128 x 128: 256 x 4096 x 4096 11.6 / 15.1 / 19.8 us, 512 x 4096 x 4096 19.5 / 16.6 / 20.8, 129 x 11008 x 4096 30.6 / 32.6 / 24.2,
// 1000 x 4096 x 4096 37.3 / 29.5 / 25.8.  Three stages (four for the smallest tile) keep the loads ahead of one work-group per compute
// unit; with more tiles than compute units two resident work-groups hide more than a third stage does, so a pair whose
// three stages do not fit twice into LDS takes two (8-bit x 8-bit, 4096^3: 85 us against 97; 3000 x 8000 x 1056: 62 against 82).
template <int FA, int FB>
static hipError_t launch_mid_pair(const TileArgs &a)
{
    constexpr int64_t CUS = 256;
    constexpr bool TWO_FIT = 3 * 4096 * ((128 * TileFmt<Fmt<FA>::bits>::ROW + 4095) / 4096 + (128 * TileFmt<Fmt<FB>::bits>::ROW + 4095) / 4096) + 8192 <= 80 * 1024;
    const int64_t m64 = (a.M + 63) / 64, m128 = (a.M + 127) / 128, n64 = (a.N + 63) / 64, n128 = (a.N + 127) / 128;
    if (m64 * n64 <= CUS) return launch_mid_t<FA, FB, 1, 1, 4>(a);
    if (m64 * n128 <= CUS) return launch_mid_t<FA, FB, 1, 2, 3>(a);
    if (TWO_FIT || m128 * n128 <= CUS) return launch_mid_t<FA, FB, 2, 2, 3>(a);
    if constexpr (!TWO_FIT) return launch_mid_t<FA, FB, 2, 2, 2>(a);
    return hipErrorNotSupported;
}

template <int FA>
static hipError_t launch_mid_a(const TileArgs &a, int fmtB)
{
    switch (fmtB) {
        case FP8_E4M3: return launch_mid_pair<FA, FP8_E4M3>(a);
        case FP8_E5M2: return launch_mid_pair<FA, FP8_E5M2>(a);
        case FP6_E3M2: return launch_mid_pair<FA, FP6_E3M2>(a);
        case FP6_E2M3: return launch_mid_pair<FA, FP6_E2M3>(a);
        default:       return launch_mid_pair<FA, FP4_E2M1>(a);
    }
}

}  // namespace mx
