// MX cast with stochastic rounding (Algorithm 1 of arXiv 2310.10537 with the element rounding
// magnitude -> step * floor(|V/X| / step + u), u = r / 2^25, r from Philox4x32-10 numbered by element),
// for both axes, every format and both source types.  Bit-identical to the generic integer kernels.
//
// Bound: the vector pipe.  A Philox call is 18 wide multiplies (a quarter of the issue rate) per four
// elements, about 0.1 ms for 2^30 of them on the chip; the rest is what the rounding itself costs.  So:
//   * each call is made once and all four words are used.  Along columns the four words belong to four
//     neighbouring columns: the lanes of a quad take every fourth row and swap words by a 4 x 4 transpose in
//     registers (two DPP exchanges).  Where the number of columns is not a multiple of four, the elements
//     of a lane start inside a call and one extra call (rows) or twice the calls (columns) cover them;
//   * the counter stays below 2^32 (larger tensors take the generic kernels), which makes two of the
//     twenty multiplies trivial and moves two more to the scalar unit; three-input xors are one
//     instruction;
//   * rounding works on whole values and the hardware converts pack them.  With s0 the smallest grid step,
//     F = floor(|V| / (X s0) * 2^25) is one multiply by a power of two and one convert.  E2M1, E2M3 and
//     INT8 values fit F into 32 bits, so the grid value is (F + (r << b)) with its low 25 + b bits cleared,
//     b the binade above the lowest two.  The wider formats round normal values directly on the Float32
//     pattern (add the top bits of r below the kept significand, clear what was discarded) and use F below
//     the smallest normal only;
//   * blocks with a non-finite value, a scale byte below 48 (above it a Float32 subnormal is less than
//     2^-25 of a step, so F = 0 gives the zero the cast asks for) or a maximum next to the Float32 limit
//     are redone with the integer encoder, one element at a time -- but not blocks of zeros, which round to
//     signed zeros under any scale: lanes outside the tensor hold them.
// A lane owns NE elements, a whole block of a large tensor and half a block of a small one (with whole blocks a
// small cast is one long chain per lane: 100 x 300 Float32 16 us along either axis, 8-10 us with halves; a large
// one gains nothing from halves, and FP6, whose convert takes 32 elements at once, loses 10 %);
// rows reach it through a wave-private LDS transpose (as in the Float32 row cast), columns through a 128 x 64 LDS
// tile (as in the column casts).
// 16384 x 2048 bf16 -> E3M2: rows 49 -> 36 us, columns 132 -> 40 us against the generic kernels; 8001 x 2050 bf16
// (both axes) 144 -> 68 us; 8001 x 2048 Float32 (both axes) 58 -> 54 us.
#include "mx_convert.hpp"
#include "mx_launch.hpp"
#include "mx_philox.hpp"

namespace mx {
namespace {

constexpr uint32_t SR_MIN_SCALE = 48;
constexpr uint32_t SR_MAX_BITS = 0x7F000000u;   // block maxima from here on take the integer encoder

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

// Philox4x32-10 for a counter below 2^32
__device__ __forceinline__ void philox32(uint32_t k0, uint32_t k1, uint32_t counter, uint32_t (&w)[4])
{
    uint32_t c0 = counter, c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
    for (int round = 0; round < 10; round++) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    w[0] = c0; w[1] = c1; w[2] = c2; w[3] = c3;
}

// words off .. off + 3 of the eight words a[0..3], b[0..3] (off = 0 .. 3)
__device__ __forceinline__ void window4(const uint32_t (&a)[4], const uint32_t (&b)[4], uint32_t off, uint32_t (&w)[4])
{
    const bool two = off & 2, one = off & 1;
    const uint32_t t0 = two ? a[2] : a[0], t1 = two ? a[3] : a[1], t2 = two ? b[0] : a[2], t3 = two ? b[1] : a[3], t4 = two ? b[2] : b[0];
    w[0] = one ? t1 : t0;
    w[1] = one ? t2 : t1;
    w[2] = one ? t3 : t2;
    w[3] = one ? t4 : t3;
}

// 4 x 4 transpose over the lanes of a quad: lane l, word m  ->  lane m, word l
__device__ __forceinline__ void quad_transpose(uint32_t (&p)[4], int ql)
{
    auto xor1 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false); };
    auto xor2 = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false); };
    const bool b0 = ql & 1, b1 = ql & 2;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const uint32_t x = p[i], y = p[i + 1], fx = xor1(x), fy = xor1(y);
        p[i] = b0 ? fy : x;
        p[i + 1] = b0 ? y : fx;
    }
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const uint32_t x = p[i], y = p[i + 2], fx = xor2(x), fy = xor2(y);
        p[i] = b1 ? fy : x;
        p[i + 2] = b1 ? y : fx;
    }
}

// log2 of the smallest grid step over X
template <int FMT> constexpr int LS0 = 1 - Fmt<FMT>::bias - Fmt<FMT>::mbits;
// largest |V| / (X s0) below 2^7: F fits 32 bits
template <int FMT> constexpr bool FITS32 = FMT == FP4_E2M1 || FMT == FP6_E2M3 || FMT == INT8;

// Four elements (Float32 patterns) onto the grid of scale byte s, with their random words.  FP formats: out is the
// signed grid value over the unit that sr_unit() names; INT8: the two's complement code in the low byte.
template <int FMT>
__device__ __forceinline__ void sr_round4(const uint32_t (&v)[4], const uint32_t (&w)[4], uint32_t s, uint32_t (&out)[4])
{
    constexpr int mb = Fmt<FMT>::mbits;
    const float c = __uint_as_float((uint32_t)(279 - LS0<FMT> - (int)s) << 23);   // 2^25 / (s0 X)
    if constexpr (FITS32<FMT>) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const float t = __builtin_fabsf(__uint_as_float(v[i])) * c;
            const uint32_t f = (uint32_t)t, r = w[i] >> 7;
            if constexpr (FMT == INT8) {
                const uint32_t q = __builtin_elementwise_add_sat(f, r) >> 25;
                const uint32_t m = (uint32_t)((int)v[i] >> 31);
                out[i] = (q ^ m) - m;
            } else {
                const int e = (int)(__float_as_uint(t) >> 23) - (127 + 25 + mb);
                const uint32_t b = (uint32_t)(e > 0 ? e : 0);
                const uint32_t g = (f + (r << b)) & (0xFE000000u << b);
                out[i] = (__float_as_uint((float)g) & 0x7FFFFFFFu) | (v[i] & 0x80000000u);
            }
        }
    } else {
        const uint32_t low = (s + 1 - Fmt<FMT>::bias) << 23;                        // smallest normal times X
        uint32_t a[4];
        uint32_t least = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            a[i] = v[i] & 0x7FFFFFFFu;
            least = least < a[i] ? least : a[i];
            out[i] = (a[i] + (w[i] >> (9 + mb))) & ~((1u << (23 - mb)) - 1u);
        }
        if (FMT == FP6_E3M2 || least < low) {       // (FP8: rare on a tensor's values)
            const float ci = __uint_as_float((uint32_t)(LS0<FMT> - 25 + (int)s) << 23);   // 1 / c
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t f = (uint32_t)(__uint_as_float(a[i]) * c);
                const uint32_t g = (f + (w[i] >> 7)) & 0xFE000000u;
                const uint32_t sub = __float_as_uint((float)g * ci);
                out[i] = a[i] < low ? sub : out[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) out[i] |= v[i] & 0x80000000u;
    }
}

// scale operand of the hardware converts for what sr_round4 returns: values over X, or over X s0 2^-25
template <int FMT>
__device__ __forceinline__ float sr_unit(uint32_t s)
{
    return FITS32<FMT> ? __uint_as_float((uint32_t)(127 + 25 - LS0<FMT>) << 23) : __uint_as_float(s << 23);
}

// NE elements of a block (all or half of it) held by a lane: value(i) = Float32 pattern of element i (registers), words(k, w) = the words of
// elements 4k .. 4k+3 (may exchange words between lanes: every lane of the wave calls it), both(x) = the larger
// x of the lanes of the block, src / stride the elements in LDS as SRC elements for the integer encoder,
// e0 / estep the numbers of its elements.  Returns the block's scale byte; packed receives NE * bits / 32 dwords.
template <int FMT, int SRC, int NE, typename V, typename W, typename B>
__device__ __forceinline__ uint32_t sr_block(V value, W words, B both, const uint8_t *src, int stride, uint64_t seed, int64_t e0,
                                             int64_t estep, uint32_t *packed)
{
    constexpr int w = Fmt<FMT>::bits, ND = NE * w / 32;
    uint32_t raw = 0, amax = 0;
#pragma unroll
    for (int i = 0; i < NE; i++) {
        const uint32_t v = value(i), a = v & 0x7FFFFFFFu;
        raw = raw > a ? raw : a;
        if (Fmt<FMT>::elem_nan) {
            const uint32_t k = amax_key<FMT>(v);
            amax = amax > k ? amax : k;
        }
    }
    raw = both(raw);
    const uint32_t s = scale_byte<FMT>(Fmt<FMT>::elem_nan ? both(amax) : raw);
    const bool fast = raw < SR_MAX_BITS && (s >= SR_MIN_SCALE || raw == 0);
    const uint32_t sq = fast && raw ? s : SR_MIN_SCALE;   // (any scale: zeros, or the block is redone below)
    const float unit = sr_unit<FMT>(sq);
    f32x16_t lo = {}, hi = {};                            // FP6: elements 2i and 2i + 1 (the convert takes 32: zeros behind half a block)
#pragma unroll
    for (int k = 0; k < NE / 4; k++) {
        uint32_t r[4], v[4], q[4];
        words(k, r);
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = value(4 * k + i);
        sr_round4<FMT>(v, r, sq, q);
        auto f = [&](int i) { return __uint_as_float(q[i]); };
        if constexpr (FMT == INT8) {
            packed[k] = (q[0] & 0xFFu) | ((q[1] & 0xFFu) << 8) | ((q[2] & 0xFFu) << 16) | (q[3] << 24);
        } else if constexpr (w == 8) {
            i16x2_t p = {0, 0};
            if (FMT == FP8_E4M3) {
                p = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(p, f(0), f(1), unit, false);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(p, f(2), f(3), unit, true);
            } else {
                p = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(p, f(0), f(1), unit, false);
                p = __builtin_amdgcn_cvt_scalef32_pk_bf8_f32(p, f(2), f(3), unit, true);
            }
            packed[k] = __builtin_bit_cast(uint32_t, p);
        } else if constexpr (w == 4) {
            uint32_t p = (k & 1) ? packed[k / 2] : 0u;
            if (k & 1) {
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, f(0), f(1), unit, 2);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, f(2), f(3), unit, 3);
            } else {
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, f(0), f(1), unit, 0);
                p = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(p, f(2), f(3), unit, 1);
            }
            packed[k / 2] = p;
        } else {
            lo[2 * k] = f(0); hi[2 * k] = f(1); lo[2 * k + 1] = f(2); hi[2 * k + 1] = f(3);
        }
    }
    if constexpr (w == 6) {
        const u32x6_t r = cvt_2xpk16_fp6_from_f32<FMT == FP6_E2M3>(lo, hi, unit);
#pragma unroll
        for (int i = 0; i < ND; i++) packed[i] = r[i];
    }
    if (!fast) {
        uint32_t o[ND];
#pragma unroll
        for (int i = 0; i < ND; i++) o[i] = 0;
        if (Fmt<FMT>::elem_nan || s != SCALE_NAN) {
#pragma unroll 1
            for (int it = 0; it < NE; it++) {
                const uint32_t v = SRC == DT_BF16 ? (uint32_t)*reinterpret_cast<const uint16_t *>(src + it * stride) << 16
                                                  : *reinterpret_cast<const uint32_t *>(src + it * stride);
                const uint32_t code = encode_elem<FMT, ROUND_STOCHASTIC>(v, s, sr_offset(seed, e0 + it * estep));
#pragma unroll
                for (int j = 0; j < ND - 1; j++) o[j] = (o[j] >> w) | (o[j + 1] << (32 - w));
                o[ND - 1] = (o[ND - 1] >> w) | (code << (32 - w));
            }
        }
#pragma unroll
        for (int i = 0; i < ND; i++) packed[i] = o[i];
    }
    return s;
}

// the codes of a block (32, 24 or 16 bytes) or of half of one
template <int w, int NE>
__device__ __forceinline__ void store_codes(uint8_t *o, const uint32_t *p)
{
    struct __attribute__((packed, aligned(4))) dword3 { uint32_t a, b, c; };
    if constexpr (NE == BLOCK) {
        if constexpr (w == 6) {
#pragma unroll
            for (int i = 0; i < 6; i += 2) *reinterpret_cast<uint2 *>(o + 4 * i) = make_uint2(p[i], p[i + 1]);
        } else {
#pragma unroll
            for (int i = 0; i < w; i += 4) st16(o + 4 * i, make_uint4(p[i], p[i + 1], p[i + 2], p[i + 3]));
        }
    } else if constexpr (w == 8) st16(o, make_uint4(p[0], p[1], p[2], p[3]));
    else if constexpr (w == 6) *reinterpret_cast<dword3 *>(o) = dword3{p[0], p[1], p[2]};
    else *reinterpret_cast<uint2 *>(o) = make_uint2(p[0], p[1]);
}

// n consecutive elements (n < N: the rest zero) as one 16-byte piece
template <int SRC>
__device__ __forceinline__ uint4 load_piece(const uint8_t *g, int n)
{
    constexpr int N = SRC == DT_BF16 ? 8 : 4;
    if (n == N) return ld16_nt(g);
    uint32_t d[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < N; i++)
        if (i < n) {
            if (SRC == DT_BF16) d[i >> 1] |= (uint32_t)reinterpret_cast<const uint16_t *>(g)[i] << (16 * (i & 1));
            else d[i] = reinterpret_cast<const uint32_t *>(g)[i];
        }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// ---------------------------------------------------------------------------------------------
// Rows.  A wave takes 64 or 32 consecutive blocks; geom counts units of 16 bytes of source.  MIS: the columns are
// not a multiple of four, so a block starts at any word of a Philox call.
// ---------------------------------------------------------------------------------------------
template <int FMT, int SRC, bool MIS, int NE>
__global__ __launch_bounds__(256) void cast_row_sr_kernel(const uint8_t *__restrict__ src, RowGeom geom, uint8_t *__restrict__ elems,
                                                          uint8_t *__restrict__ scales, uint64_t seed)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits, ESZ = SRC == DT_BF16 ? 2 : 4, EPU = 16 / ESZ, UPL = NE / EPU;   // UPL: 16-byte pieces per lane
    constexpr int PITCH = NE * ESZ + 16;               // bytes per lane in LDS: 16-byte reads of 16 lanes cover all banks
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * 64 * PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint8_t *lds = lds_all + wave * 64 * PITCH;
    const uint32_t lane0 = (blockIdx.x * 4 + wave) * 64, u0 = lane0 * UPL;
    if (u0 >= geom.n_units) return;
    uint4 d[UPL];
#pragma unroll
    for (int j = 0; j < UPL; j++) {
        const uint32_t u = u0 + j * 64 + lane;
        d[j] = make_uint4(0, 0, 0, 0);
        if (u < geom.n_units) {
            int n;
            const int64_t at = geom.at(u, EPU, n);
            if (n > 0) d[j] = load_piece<SRC>(src + at * ESZ, n);
        }
    }
#pragma unroll
    for (int j = 0; j < UPL; j++) {
        const int q = j * 64 + lane;
        *reinterpret_cast<uint4 *>(lds + (q / UPL) * PITCH + (q % UPL) * 16) = d[j];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);                  // lgkmcnt(0): the wave's own LDS writes
    __builtin_amdgcn_wave_barrier();
    const uint8_t *mine = lds + lane * PITCH;
    uint32_t x[UPL * 4];
#pragma unroll
    for (int j = 0; j < UPL; j++) {
        const uint4 t = *reinterpret_cast<const uint4 *>(mine + 16 * j);
        x[4 * j] = t.x; x[4 * j + 1] = t.y; x[4 * j + 2] = t.z; x[4 * j + 3] = t.w;
    }
    // number of the first element in the tensor (rows without the fill)
    const uint32_t ub = (lane0 + lane) * UPL, r = geom.units_per_row(ub);
    const int64_t e0 = (int64_t)r * geom.cols + (int64_t)(ub - r * geom.units_per_row.d) * EPU;
    const uint32_t ctr = (uint32_t)(e0 >> 2), off = (uint32_t)e0 & 3u;
    uint32_t next[4];
    if (MIS) philox32((uint32_t)seed, (uint32_t)(seed >> 32), ctr, next);
    uint32_t packed[NE * w / 32];
    const uint32_t s = sr_block<FMT, SRC, NE>(
        [&](int i) { return SRC == DT_F32 ? x[i] : (i & 1) ? x[i >> 1] & 0xFFFF0000u : x[i >> 1] << 16; },
        [&](int k, uint32_t (&rw)[4]) {
            if constexpr (MIS) {
                uint32_t cur[4] = {next[0], next[1], next[2], next[3]};
                philox32((uint32_t)seed, (uint32_t)(seed >> 32), ctr + (uint32_t)k + 1u, next);
                window4(cur, next, off, rw);
            } else {
                philox32((uint32_t)seed, (uint32_t)(seed >> 32), ctr + (uint32_t)k, rw);
            }
        },
        [](uint32_t v) { return group_max<BLOCK / NE>(v); }, mine, ESZ, seed, e0, 1, packed);
    if (ub >= geom.n_units) return;
    store_codes<w, NE>(elems + (int64_t)(lane0 + lane) * (NE * w / 8), packed);
    if (NE == BLOCK || !(lane & 1)) scales[(lane0 + lane) / (BLOCK / NE)] = (uint8_t)s;
}

// ---------------------------------------------------------------------------------------------
// Columns.  Tile 128 rows x 64 columns, four waves (eight with halves); lane -> column (t & 3) + 4 (t / 16), block (t / 4) % 4: the
// four lanes of a quad hold four neighbouring columns of the same rows, i.e. the four words of a call per row.
// ---------------------------------------------------------------------------------------------
constexpr int SR_R = 128, SR_C = 64;
template <int FMT, int SRC, bool MIS, int NE>
__global__ __launch_bounds__(SR_R / NE * SR_C) void cast_col_sr_kernel(const uint8_t *__restrict__ src, int64_t rows, int64_t cols, int64_t ld,
                                                          uint8_t *__restrict__ elems, uint8_t *__restrict__ scales, int64_t row_tiles,
                                                          int64_t n_tiles, int64_t per_xcd, uint64_t seed)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits, ESZ = SRC == DT_BF16 ? 2 : 4, EPU = 16 / ESZ, PARTS = SR_R / NE, THREADS = PARTS * SR_C;
    constexpr int PITCH = SR_C * ESZ, ROT = 64 / PARTS * ESZ;   // row parts rotated against each other: conflict-free column reads
    __shared__ __attribute__((aligned(16))) uint8_t tile[SR_R * PITCH];
    const int t = threadIdx.x;
    const int64_t tile_id = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || tile_id >= n_tiles) return;   // uniform over the work-group
    const int64_t c0 = tile_id / row_tiles * SR_C, r0 = tile_id % row_tiles * SR_R;
    {
        constexpr int LPR = SR_C / EPU, RPP = THREADS / LPR, NP = SR_R / RPP;
        const int lr = t / LPR, lc = t % LPR;
        const int64_t left = cols - c0 - lc * EPU;
        const int n = left >= EPU ? EPU : left > 0 ? (int)left : 0;
        uint4 v[NP];
#pragma unroll
        for (int p = 0; p < NP; p++) {
            v[p] = make_uint4(0, 0, 0, 0);
            const int64_t row = r0 + p * RPP + lr;
            if (n > 0 && row < rows) v[p] = load_piece<SRC>(src + (row * ld + c0 + lc * EPU) * ESZ, n);
        }
#pragma unroll
        for (int p = 0; p < NP; p++) {
            const int r = p * RPP + lr;
            *reinterpret_cast<uint4 *>(tile + r * PITCH + ((lc * 16 + (r / NE) * ROT) & (PITCH - 1))) = v[p];
        }
    }
    __syncthreads();
    const int ql = t & 3, c = ql + t / (4 * PARTS) * 4, hb = (t >> 2) % PARTS;
    const uint8_t *mine = tile + hb * NE * PITCH + ((c * ESZ + hb * ROT) & (PITCH - 1));
    constexpr int NX = SRC == DT_BF16 ? NE / 2 : NE;
    uint32_t x[NX];
#pragma unroll
    for (int i = 0; i < NX; i++) {
        if (SRC == DT_BF16)
            x[i] = *reinterpret_cast<const uint16_t *>(mine + 2 * i * PITCH) | ((uint32_t)*reinterpret_cast<const uint16_t *>(mine + (2 * i + 1) * PITCH) << 16);
        else
            x[i] = *reinterpret_cast<const uint32_t *>(mine + i * PITCH);
    }
    // first element of the quad's columns in this lane's first row (row ql of its part)
    const int64_t eq = (r0 + hb * NE + ql) * cols + c0 + (c & ~3);
    uint32_t packed[NE * w / 32];
    const uint32_t s = sr_block<FMT, SRC, NE>(
        [&](int i) { return SRC == DT_F32 ? x[i] : (i & 1) ? x[i >> 1] & 0xFFFF0000u : x[i >> 1] << 16; },
        [&](int k, uint32_t (&rw)[4]) {
            if constexpr (MIS) {
                const int64_t e = eq + 4 * k * cols;
                uint32_t a[4], b[4];
                philox32((uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)(e >> 2), a);
                philox32((uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)(e >> 2) + 1u, b);
                window4(a, b, (uint32_t)e & 3u, rw);
            } else {
                philox32((uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)(eq >> 2) + (uint32_t)k * (uint32_t)cols, rw);
            }
            quad_transpose(rw, ql);
        },
        [](uint32_t v) {
            if (NE == BLOCK) return v;
            const uint32_t o = (uint32_t)__shfl_xor((int)v, 4);
            return v > o ? v : o;
        }, mine, PITCH, seed,
        (r0 + hb * NE) * cols + c0 + c, cols, packed);
    const int64_t n_rb = (rows + BLOCK - 1) / BLOCK, row_blk = r0 / BLOCK + hb / (BLOCK / NE);
    if (c0 + c >= cols || row_blk >= n_rb) return;
    const int64_t blk = (c0 + c) * n_rb + row_blk;
    store_codes<w, NE>(elems + blk * (BLOCK * w / 8) + (hb % (BLOCK / NE)) * (NE * w / 8), packed);
    if (hb % (BLOCK / NE) == 0) scales[blk] = (uint8_t)s;
}

template <int FMT, int SRC, int NE>
hipError_t launch_sr_ne(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems, uint8_t *scales, uint64_t seed,
                     hipStream_t st)
{
    const uint8_t *p = static_cast<const uint8_t *>(src);
    constexpr int EPU = SRC == DT_BF16 ? 8 : 4;
    const int64_t pcols = (cols + BLOCK - 1) / BLOCK * BLOCK, prows = (rows + SR_R - 1) / SR_R * SR_R;
    // element numbers below 2^34 (32-bit Philox counters, the padding of the last tile and call included)
    if ((double)prows * (double)(pcols + 64) >= 17179869184.0) return hipErrorNotSupported;
    if (axis == 1) {
        const int64_t units = rows * (pcols / EPU);
        if (units > 0x7FFFFFFF) return hipErrorNotSupported;
        const RowGeom geom = row_geom(1, rows, cols, ld, rows * ld, EPU);
        const dim3 grid((unsigned)((rows * (pcols / NE) + 255) / 256));
        if (cols & 3) hipLaunchKernelGGL((cast_row_sr_kernel<FMT, SRC, true, NE>), grid, dim3(256), 0, st, p, geom, elems, scales, seed);
        else hipLaunchKernelGGL((cast_row_sr_kernel<FMT, SRC, false, NE>), grid, dim3(256), 0, st, p, geom, elems, scales, seed);
        return hipGetLastError();
    }
    const int64_t row_tiles = prows / SR_R, n_tiles = row_tiles * ((cols + SR_C - 1) / SR_C), per_xcd = (n_tiles + 7) / 8;
    if (per_xcd * 8 > 0x7FFFFFFF) return hipErrorNotSupported;
    const dim3 grid((unsigned)(per_xcd * 8));
    if (cols & 3)
        hipLaunchKernelGGL((cast_col_sr_kernel<FMT, SRC, true, NE>), grid, dim3(SR_R / NE * SR_C), 0, st, p, rows, cols, ld, elems, scales, row_tiles, n_tiles,
                           per_xcd, seed);
    else
        hipLaunchKernelGGL((cast_col_sr_kernel<FMT, SRC, false, NE>), grid, dim3(SR_R / NE * SR_C), 0, st, p, rows, cols, ld, elems, scales, row_tiles, n_tiles,
                           per_xcd, seed);
    return hipGetLastError();
}

// whole blocks per lane once they give every SIMD several waves (2^24 elements: eight)
template <int FMT, int SRC>
hipError_t launch_sr(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems, uint8_t *scales, uint64_t seed,
                     hipStream_t st)
{
    return rows * cols >= ((int64_t)1 << 24) ? launch_sr_ne<FMT, SRC, BLOCK>(src, rows, cols, ld, axis, elems, scales, seed, st)
                                             : launch_sr_ne<FMT, SRC, BLOCK / 2>(src, rows, cols, ld, axis, elems, scales, seed, st);
}

template <int SRC>
hipError_t launch_sr_fmt(int fmt, const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems, uint8_t *scales,
                         uint64_t seed, hipStream_t st)
{
    switch (fmt) {
        case FP8_E4M3: return launch_sr<FP8_E4M3, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
        case FP8_E5M2: return launch_sr<FP8_E5M2, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
        case FP6_E3M2: return launch_sr<FP6_E3M2, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
        case FP6_E2M3: return launch_sr<FP6_E2M3, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
        case FP4_E2M1: return launch_sr<FP4_E2M1, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
        default:       return launch_sr<INT8, SRC>(src, rows, cols, ld, axis, elems, scales, seed, st);
    }
}

}  // namespace

hipError_t launch_cast_sr(const void *src, int src_dt, int64_t rows, int64_t cols, int64_t ld, int axis, int fmt, uint64_t seed,
                          uint8_t *elems, uint8_t *scales, hipStream_t st)
{
    return src_dt == DT_BF16 ? launch_sr_fmt<DT_BF16>(fmt, src, rows, cols, ld, axis, elems, scales, seed, st)
                             : launch_sr_fmt<DT_F32>(fmt, src, rows, cols, ld, axis, elems, scales, seed, st);
}

}  // namespace mx
