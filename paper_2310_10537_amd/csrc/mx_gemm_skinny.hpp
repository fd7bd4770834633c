// MX GEMM (Section 4.1 of arXiv 2310.10537) for few rows of A -- the shape of a decoding step,
// where the time goes into streaming the weight operand B once.
//
// The direct kernel gives such a problem one wave per 32 x 32 output tile and lets it walk the
// whole K range alone, one load-then-multiply after the other: with N / 32 waves on the chip and
// every step paying a full memory latency, 4096 x 4096 weights take 25-45 us (0.4-0.7 TB/s).  Here a
// work-group of eight waves owns 32 columns of C and all (up to 128) rows: the K range is cut into
// eight contiguous slices, one per wave, each wave requests the operands of several K steps before
// it multiplies the first, and the eight partial sums meet in LDS in a fixed order (so the result
// does not depend on timing).  B is read exactly once; A, a few KB per K step, comes from L2.
#pragma once

#include "mx_gemm_tile.hpp"
#include "mx_convert.hpp"

namespace mx {

constexpr int SK_WAVES = 8;
constexpr int64_t SK_MAX_K = (int64_t)1 << 25;       // of the staged kernel

// ---------------------------------------------------------------------------------------------
// K a multiple of 128: operands staged through LDS.
// In the kernel further down every lane of an operand load addresses a different matrix row, so
// a load instruction touches 32 cache lines and a compute unit makes eight line accesses for every
// line it needs: that, not bandwidth or latency, bounds it (9.4 us for 4096 x 4096 weights at
// M = 1).  Here each wave fetches its slice 128 elements at a time with loads whose adjacent lanes
// read adjacent 16 bytes of a row (every line touched once), parks the 16-byte pieces in a private
// LDS tile laid out exactly as the large tiled kernel lays out its stages (same swizzles, same
// operand reads), and multiplies from there; the next chunk's loads are in flight meanwhile.
// Rows beyond M and columns beyond N read a valid row instead (clamped), as every load of a step then sits in one straight run that
// the waits can count; such results are never stored.  (A branch per load to leave absent rows out made every wait one for all
// loads in flight: 9 x 5120 x 7424 E4M3 8.8 us clamped, 15.9 with branches; 32 x 2503 x 17536 24.7 and 40.6; 64 rows 10 % slower.)
// Up to 8 or 16 rows A has loads of its own.  The load path takes its time by the line touched, 2.6 to 3.2 clocks each, whole or
// not: with the loads of 32 rows A's pieces of a chunk were 48 such lines against 16 of 4-bit weights.  Against those two chunks of A go
// together as well (PAIR_A): whole lines of 4- and 8-bit rows, two lines instead of three of 6-bit ones, and one wait instead of two.
// 16 x 28672 x 8192 E3M2 x E2M1 36.2 us with the loads of 32 rows, 31.8 so (4 TB/s of weights); 16 x 4096 x 14336 12.2 / 10.1; 12 x 4096 x 4096
// E4M3 pairs 6.5 / 6.1; 1 x 16128 x 8192 E4M3 x E2M1, 8 rows in both, 13.7 / 13.2 from the pairs alone.  The second chunk's 16 rows take the
// tile's place of rows 16 .. 31, so 17 rows and more go a chunk at a time.
// 4-bit B, up to 32 rows: two chunks at a time, 128 bytes of a row -- whole lines -- in flight for two steps; and the scales of four
// chunks in one 16-byte load per row, which waits in LDS for its chunks: a dword per chunk touches each line four times as often, in
// a cache that B streams through.  16 x 28672 x 8192 E3M2 x E2M1, weights from HBM: a chunk and a dword at a time 49.8 us, two
// chunks 43.0, with the groups 36.4.
// No bound on the registers: 128 would always let two work-groups share a compute unit, but made 38 of the 100 cast-on-load instances spill.
// QA: up to 16 rows of bf16 activations are cast on load -- a lane takes one block of a chunk and parks its codes, the
// same cast and hence the same bytes as the stand-alone one.
// ---------------------------------------------------------------------------------------------
template <int W> struct SkStage {                    // one 32-row block of a 128-element chunk
    static constexpr int NJ = W == 4 ? 2 : 4;        // loads per lane: 16 (4-bit) or 8 rows per wave-wide load
    static constexpr int BYTES = 32 * TileFmt<W>::ROW;
};

constexpr int MX_OPERAND = -1;                       // QA: A is an MX operand, else the rounding of its cast
// ROWS: the most rows an MX operand A has, 8, 16 or 32 * MT
template <int FA, int FB, int MT, int CDT, int QA = MX_OPERAND, int ROWS = 32 * MT>
__global__ __launch_bounds__(64 * SK_WAVES, 1) void gemm_skinny_lds_kernel(int64_t M, int64_t N, int64_t K,
                                                                         const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                                                         const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                                         void *__restrict__ C, int64_t ldc, int64_t lda)
{
    constexpr bool CAST = QA != MX_OPERAND;          // A: bf16 [M][lda], at most 16 rows
    static_assert(MT == 1 || (!CAST && ROWS == 32 * MT), "one 32-row tile");
    constexpr int WA = Fmt<FA>::bits, WB = Fmt<FB>::bits;
    constexpr int HA = hw_fmt(FA), HB = hw_fmt(FB);   // must reach the builtin as literal constants
    constexpr int CB = MT == 1 && WB == 4 ? 2 : 1;    // chunks of B loaded together
    constexpr bool PAIR_A = CB == 2 && ROWS <= 16 && !CAST;     // two chunks of A loaded together
    constexpr bool GROUPS = CB == 2;                  // scales of four chunks in one load, by way of LDS
    constexpr int A_BYTES = MT * SkStage<WA>::BYTES, B_BYTES = CB * SkStage<WB>::BYTES, W_BYTES = A_BYTES + B_BYTES + (GROUPS ? 1024 : 0);
    constexpr int RED_BYTES = (SK_WAVES - 1) * MT * 16 * 64 * 4;
    constexpr int LDS_BYTES = SK_WAVES * W_BYTES > RED_BYTES ? SK_WAVES * W_BYTES : RED_BYTES;
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, i = lane & 31, g = lane >> 5;
    const int64_t n0 = (int64_t)blockIdx.x * 32, m0 = (int64_t)blockIdx.y * (32 * MT);
    const int64_t nkb = K / BLOCK, chunks = K / 128;
    const int64_t per_wave = (chunks + SK_WAVES - 1) / SK_WAVES;
    const int64_t c_begin = wave * per_wave, c_end = c_begin + per_wave < chunks ? c_begin + per_wave : chunks;
    uint8_t *tA = lds + wave * W_BYTES, *tB = tA + A_BYTES;

    // ---- staging: lane -> (row l / P, 16-byte piece l % P) of a wave-wide load; P pieces per row chunk
    // PAIR_A: the P = 2 WA pieces of both chunks in a row, a run of 64 after the other; the second chunk's tile stands where rows 16 .. 31 would be
    constexpr int PA = PAIR_A ? 2 * WA : WA == 4 ? 4 : 8, PB = WB == 4 ? 4 * CB : 8;       // (6-bit: pieces 6 and 7 stay idle)
    constexpr int NJA = ((ROWS < 32 ? ROWS : 32) * PA + 63) / 64, NJB = CB * SkStage<WB>::NJ;
    const int ar = lane / PA, ap = lane % PA, br = lane / PB, bp = lane % PB;
    const bool a_on = PAIR_A || WA != 6 || ap < 6, b_on = WB != 6 || bp < 6;
    const int64_t a_rb = K * WA / 8, b_rb = K * WB / 8;                   // bytes per matrix row
    auto clampi = [](int64_t v, int64_t hi) { return v < hi ? v : hi; };
    // 32-bit offsets of the lane's pieces from wave-uniform addresses (K up to SK_MAX_K: 127 rows stay below 2^32 bytes)
    uint32_t a_ofs[MT][NJA], b_ofs[NJB];
#pragma unroll
    for (int x = 0; x < MT; x++)
#pragma unroll
        for (int j = 0; j < NJA; j++) {
            const int n = j * 64 + lane, r = PAIR_A ? n / PA : j * (64 / PA) + ar, p = PAIR_A ? n % PA : ap;
            a_ofs[x][j] = (uint32_t)clampi(32 * x + r, M - 1 - m0) * (uint32_t)a_rb + p * 16;
        }
#pragma unroll
    for (int j = 0; j < NJB; j++) b_ofs[j] = (uint32_t)clampi(j * (64 / PB) + br, N - 1 - n0) * (uint32_t)b_rb + bp * 16;
    uint32_t sa_ofs[MT];
    const uint32_t sb_ofs = (uint32_t)clampi(i, N - 1 - n0) * (uint32_t)nkb;
#pragma unroll
    for (int x = 0; x < MT; x++) sa_ofs[x] = (uint32_t)clampi(32 * x + i, M - 1 - m0) * (uint32_t)nkb;
    // A wave-uniform address and a 32-bit offset per lane, kept apart up to the load (the empty asm statements hide them from the
    // loop optimiser): it would carry a 64-bit address per load instead -- with 128 rows 50 vector registers, and 8-bit operands spill
    // (512 x 128 x 3456 E4M3 21.7 us, 16.5 so).  Up to 32 rows there is room for them, and one add less per load measured 5-10 % faster.
    typedef const __attribute__((address_space(1))) uint8_t *global_ptr;
    auto scalar = [](const uint8_t *p) {
        global_ptr g = (global_ptr)p;
        if constexpr (MT > 1) asm volatile("" : "+s"(g));
        return g;
    };
    auto piece = [](global_ptr p, uint32_t o) {           // 16 bytes
        if constexpr (MT > 1) asm volatile("" : "+v"(o));
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 v = *(const __attribute__((address_space(1))) u32x4 *)(p + o);
        return make_uint4(v.x, v.y, v.z, v.w);
    };
    auto dword = [](global_ptr p, uint32_t o) {
        if constexpr (MT > 1) asm volatile("" : "+v"(o));
        return *(const __attribute__((address_space(1))) uint32_t *)(p + o);
    };
    auto lds_slot = [](int w, int r, int c) {
        return w == 8 ? r * 128 + ((c ^ ((r >> 1) & 7)) << 4) : w == 6 ? r * 96 + ((c ^ ((r >> 3) & 1)) << 4)
                                                                       : r * 64 + ((c ^ ((r >> 2) & 3)) << 4);
    };
    uint4 ra[MT][NJA], rq[4], rb[NJB];
    uint32_t sa_d[MT], sb_d;
    const int qr = lane >> 2, qb = lane & 3;          // CAST: the lane's row and its block of a chunk
    const uint8_t *const q0 = Ae + (qr * lda + qb * 32) * 2;              // (dereferenced where the row exists)
    auto request_a = [&](int64_t c) {
        if constexpr (CAST) {
            if (qr < M) {
#pragma unroll
                for (int j = 0; j < 4; j++) rq[j] = ld16(q0 + c * 256 + j * 16);
            }
        } else {
            const global_ptr p = scalar(Ae + m0 * a_rb + c * (128 * WA / 8));
            if (a_on) {
#pragma unroll
                for (int x = 0; x < MT; x++)
#pragma unroll
                    for (int j = 0; j < NJA; j++) {           // (a second chunk beyond K: the first one again)
                        const uint32_t back = PAIR_A && c + 1 >= chunks && (j * 64 + lane) % PA >= WA ? 16 * WA : 0;
                        ra[x][j] = piece(p, a_ofs[x][j] - back);
                    }
            }
        }
    };
    auto request_b = [&](int64_t c) {                                     // (a second chunk beyond K: the first one again)
        const global_ptr p = scalar(Be + n0 * b_rb + c * (128 * WB / 8));
        const uint32_t back = CB == 2 && bp >= 4 && c + 1 >= chunks ? 64 : 0;
        if (b_on) {
#pragma unroll
            for (int j = 0; j < NJB; j++) rb[j] = piece(p, b_ofs[j] - back);
        }
    };
    // GROUPS: lanes 0 .. 31 fetch the scale bytes of rows of A, lanes 32 .. 63 of B (CAST: all of B); the last group of a row is
    // its last 16 bytes and sits further back in the slot
    uint8_t *const tS = tB + B_BYTES;
    const uint8_t *const srow = g == 0 && !CAST ? As + (m0 + clampi(i, M - 1 - m0)) * nkb : Bs + (n0 + clampi(i, N - 1 - n0)) * nkb;
    uint4 sg = make_uint4(0, 0, 0, 0);
    auto group_at = [&](int64_t c) { return c + 4 <= chunks ? c : chunks >= 4 ? chunks - 4 : c; };
    auto request_g = [&](int64_t c) {
        if (chunks >= 4) __builtin_memcpy(&sg, __builtin_assume_aligned(srow + group_at(c) * 4, 4), 16);
        else sg.x = *reinterpret_cast<const uint32_t *>(srow + c * 4);             // fewer than four chunks: one per wave
    };
    auto request_s = [&](int64_t c) {
        if constexpr (!CAST) {
            const global_ptr p = scalar(As + m0 * nkb + c * 4);
#pragma unroll
            for (int x = 0; x < MT; x++) sa_d[x] = dword(p, sa_ofs[x]);
        }
        sb_d = dword(scalar(Bs + n0 * nkb + c * 4), sb_ofs);
    };
    uint8_t *const cast_sc = tA + 16 * TileFmt<WA>::ROW;                  // CAST: the scales of 16 rows, where rows 16 .. 31 would be
    auto park_a = [&]() {
        if constexpr (CAST) {
            // on for the converts only: matrix instructions would clamp NaN / Inf operands of B and results
            if constexpr (FA == FP8_E4M3 || FA == FP8_E5M2) fp8_saturate_mode(true);
            if (qr < M) {
                uint32_t d[16], out[WA];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    d[4 * j] = rq[j].x; d[4 * j + 1] = rq[j].y; d[4 * j + 2] = rq[j].z; d[4 * j + 3] = rq[j].w;
                }
                cast_sc[lane] = (uint8_t)quantize_block_bf16<FA, QA>(d, out);
#pragma unroll
                for (int q = 0; q < WA / 2; q++) {
                    const int o = qb * (4 * WA) + 8 * q;                      // byte of the row's chunk
                    *reinterpret_cast<uint2 *>(tA + lds_slot(WA, qr, o >> 4) + (o & 15)) = make_uint2(out[2 * q], out[2 * q + 1]);
                }
            }
            if constexpr (FA == FP8_E4M3 || FA == FP8_E5M2) fp8_saturate_mode(false);
        } else if constexpr (PAIR_A) {
#pragma unroll
            for (int j = 0; j < NJA; j++) {
                const int n = j * 64 + lane, r = n / PA, p = n % PA;
                if (ROWS * PA % 64 == 0 || n < ROWS * PA)
                    *reinterpret_cast<uint4 *>(tA + (p >= WA ? A_BYTES / 2 + lds_slot(WA, r, p - WA) : lds_slot(WA, r, p))) = ra[0][j];
            }
        } else if (a_on) {
#pragma unroll
            for (int x = 0; x < MT; x++)
#pragma unroll
                for (int j = 0; j < NJA; j++)
                    *reinterpret_cast<uint4 *>(tA + x * SkStage<WA>::BYTES + lds_slot(WA, j * (64 / PA) + ar, ap)) = ra[x][j];
        }
    };
    auto park_b = [&]() {
        if (b_on) {
#pragma unroll
            for (int j = 0; j < NJB; j++)
                *reinterpret_cast<uint4 *>(tB + (CB == 2 ? (bp >> 2) * SkStage<WB>::BYTES + lds_slot(WB, j * (64 / PB) + br, bp & 3)
                                                         : lds_slot(WB, j * (64 / PB) + br, bp))) = rb[j];
        }
    };
    const FragOfs<WA> fa = frag_ofs<WA>(i, g);
    const FragOfs<WB> fb = frag_ofs<WB>(i, g);

    v16f_t acc[MT];
#pragma unroll
    for (int x = 0; x < MT; x++)
#pragma unroll
        for (int t = 0; t < 16; t++) acc[x][t] = 0.f;

    if (c_begin < c_end) {
        if constexpr (GROUPS) request_g(c_begin);
        request_a(c_begin);
        request_b(c_begin);
        if constexpr (!GROUPS) request_s(c_begin);
    }
    int pos = 0;                                      // GROUPS: the chunk's dword in its group's slot
    for (int64_t c0 = c_begin; c0 < c_end; c0 += CB) {
        if constexpr (GROUPS) {
            if (((c0 - c_begin) & 3) == 0) {
                *reinterpret_cast<uint4 *>(tS + lane * 16) = sg;
                pos = (int)(c0 - group_at(c0));
                if (c0 + 4 < c_end) request_g(c0 + 4);
            }
        }
#pragma unroll
        for (int k = 0; k < CB; k++) {
            const int64_t c = c0 + k;
            if (k > 0 && c >= c_end) break;
            if (!PAIR_A || k == 0) park_a();
            if (k == 0) park_b();
            uint32_t sa[MT], sb;
            if constexpr (!GROUPS) {
#pragma unroll
                for (int x = 0; x < (CAST ? 0 : MT); x++) sa[x] = sa_d[x];
                sb = sb_d;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
            if constexpr (GROUPS) {
                if constexpr (!CAST) sa[0] = *reinterpret_cast<const uint32_t *>(tS + i * 16 + pos * 4);
                sb = *reinterpret_cast<const uint32_t *>(tS + 512 + i * 16 + pos * 4);
                pos++;
            }
            if constexpr (CAST) sa[0] = reinterpret_cast<const uint32_t *>(cast_sc)[i & 15];
            // lanes 32 .. 63 shift their scale dword by a byte: one selector then addresses block 2 sub + g
            sb = g ? sb >> 8 : sb;
#pragma unroll
            for (int x = 0; x < MT; x++) sa[x] = g ? sa[x] >> 8 : sa[x];
            // loads return in order: the scales, wanted last, behind the operands of their step
            if (!PAIR_A && c + 1 < c_end) request_a(c + 1);
            if (PAIR_A && k == 0 && c0 + CB < c_end) request_a(c0 + CB);
            if (CB == 1 && c + 1 < c_end) request_b(c + 1);
            if (!GROUPS && c + 1 < c_end) request_s(c + 1);
            if (CB == 2 && k == 0 && c0 + CB < c_end) request_b(c0 + CB);
            const uint8_t *tb = tB + k * SkStage<WB>::BYTES, *ta = tA + (PAIR_A ? k * (A_BYTES / 2) : 0);
            const v8i_t b0 = read_frag<WB>(tb, fb, 0, 0), b1 = read_frag<WB>(tb, fb, 1, 0);
#pragma unroll
            for (int x = 0; x < MT; x++) {
                const v8i_t a0 = read_frag<WA>(ta + x * SkStage<WA>::BYTES, fa, 0, 0), a1 = read_frag<WA>(ta + x * SkStage<WA>::BYTES, fa, 1, 0);
                acc[x] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a0, b0, acc[x], HA, HB, 0, (int)sa[x], 0, (int)sb);
                acc[x] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a1, b1, acc[x], HA, HB, 2, (int)sa[x], 2, (int)sb);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the tile is read before the next chunk is parked in it
            __builtin_amdgcn_wave_barrier();
        }
    }

    // ---- the eight partial sums, always w0 + w1 + ... + w7; the staging tiles are done with
    __syncthreads();
    float *red = reinterpret_cast<float *>(lds);
    if (wave > 0) {
#pragma unroll
        for (int x = 0; x < MT; x++)
#pragma unroll
            for (int t = 0; t < 16; t++) red[(((wave - 1) * MT + x) * 16 + t) * 64 + lane] = acc[x][t];
    }
    __syncthreads();
    if (wave != 0) return;
    const int64_t col = n0 + i;
#pragma unroll
    for (int x = 0; x < MT; x++)
#pragma unroll
        for (int t = 0; t < 16; t++) {
            float v = acc[x][t];
#pragma unroll
            for (int w = 0; w < SK_WAVES - 1; w++) v += red[((w * MT + x) * 16 + t) * 64 + lane];
            const int64_t r = m0 + 32 * x + 8 * (t / 4) + 4 * g + (t % 4);   // result register t: row 8 (t/4) + 4g + t%4, column i
            if (r < M && col < N) {
                if (CDT == DT_F32) reinterpret_cast<float *>(C)[r * ldc + col] = v;
                else reinterpret_cast<uint16_t *>(C)[r * ldc + col] = (uint16_t)f32_to_bf16_bits(v);
            }
        }
}

}  // namespace mx
