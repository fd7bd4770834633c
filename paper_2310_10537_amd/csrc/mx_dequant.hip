// MX dequantize kernels: v = X * P (Section 2 of arXiv 2310.10537) for gfx950.
// One lane turns 8 consecutive element codes of a block (w bytes) into 8 values.
#include "mx_device.hpp"
#include "mx_launch.hpp"

namespace mx {

// 8 codes = w bytes starting at a w-byte-aligned address
template <int FMT>
__device__ __forceinline__ void load_codes8(const uint8_t *p, uint32_t (&c)[8])
{
    constexpr int w = Fmt<FMT>::bits;
    uint64_t bits;
    if (w == 8) {
        uint2 d = *reinterpret_cast<const uint2 *>(p);
        bits = (uint64_t)d.x | ((uint64_t)d.y << 32);
    } else if (w == 4) {
        bits = *reinterpret_cast<const uint32_t *>(p);
    } else {
        const uint16_t *h = reinterpret_cast<const uint16_t *>(p);
        bits = (uint64_t)h[0] | ((uint64_t)h[1] << 16) | ((uint64_t)h[2] << 32);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) c[i] = (uint32_t)(bits >> (w * i)) & ((1u << w) - 1u);
}

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x32_t __attribute__((ext_vector_type(32)));
typedef uint32_t u32x6_t_ __attribute__((ext_vector_type(6)));
typedef __bf16 bf16x2_t_ __attribute__((ext_vector_type(2)));

// 8 consecutive codes (w bytes at p) times X = 2^(s-127) as Float32, with gfx950's scaled
// up-converts (V_CVT_SCALEF32_PK_F32_FP8 / _BF8 / _FP4, _PK32_F32_FP6 / _BF6): checked against the
// CPU reference for every code at every scale byte 0 .. 254 -- subnormal codes, NaN and Inf
// codes, products that overflow Float32 and X = 2^-127 included -- they return exactly X * P.
// (The integer decode costs about 20 vector instructions per element, which made the kernel
// compute-bound.)  The NaN scale 0xFF is the caller's business.
template <int FMT>
__device__ __forceinline__ void decode8_hw(const uint8_t *p, uint32_t s, float (&f)[8])
{
    const float sf = __uint_as_float(s << 23);
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) {
        const uint2 d = *reinterpret_cast<const uint2 *>(p);
        const uint32_t dw[2] = {d.x, d.y};
#pragma unroll
        for (int j = 0; j < 2; j++) {
            f32x2_t lo, hi;
            if (FMT == FP8_E4M3) {
                lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(dw[j], sf, false);
                hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(dw[j], sf, true);
            } else {
                lo = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(dw[j], sf, false);
                hi = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(dw[j], sf, true);
            }
            f[4 * j] = lo[0]; f[4 * j + 1] = lo[1]; f[4 * j + 2] = hi[0]; f[4 * j + 3] = hi[1];
        }
    } else if constexpr (FMT == FP4_E2M1) {
        const uint32_t d = *reinterpret_cast<const uint32_t *>(p);
#pragma unroll
        for (int j = 0; j < 4; j++) {
            f32x2_t v;
            if (j == 0) v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(d, sf, 0);
            if (j == 1) v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(d, sf, 1);
            if (j == 2) v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(d, sf, 2);
            if (j == 3) v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(d, sf, 3);
            f[2 * j] = v[0]; f[2 * j + 1] = v[1];
        }
    } else if constexpr (FMT == FP6_E3M2 || FMT == FP6_E2M3) {
        // 8 codes = 48 bits; the 32-element convert takes them in the low bits of its six dwords
        const uint16_t *h = reinterpret_cast<const uint16_t *>(p);
        const u32x6_t_ d = {(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2], 0u, 0u, 0u, 0u};
        const f32x32_t v = FMT == FP6_E2M3 ? __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(d, sf)
                                           : __builtin_amdgcn_cvt_scalef32_pk32_f32_bf6(d, sf);
#pragma unroll
        for (int i = 0; i < 8; i++) f[i] = v[i];
    }
}

// 8 codes already in registers (lo: the first 32 bits of the w-byte unit, hi: the rest) times X
template <int FMT>
__device__ __forceinline__ void decode8_regs(uint32_t lo, uint32_t hi, uint32_t s, float (&f)[8])
{
    constexpr int w = Fmt<FMT>::bits;
    if (FMT == INT8 || s == SCALE_NAN) {
        const uint64_t bits = (uint64_t)lo | ((uint64_t)hi << 32);
#pragma unroll
        for (int i = 0; i < 8; i++) f[i] = decode_scaled<FMT>((uint32_t)(bits >> (w * i)) & ((1u << w) - 1u), s);
        return;
    }
    const float sf = __uint_as_float(s << 23);
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) {
        const uint32_t dw[2] = {lo, hi};
#pragma unroll
        for (int j = 0; j < 2; j++) {
            f32x2_t a, b;
            if (FMT == FP8_E4M3) {
                a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(dw[j], sf, false);
                b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(dw[j], sf, true);
            } else {
                a = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(dw[j], sf, false);
                b = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(dw[j], sf, true);
            }
            f[4 * j] = a[0]; f[4 * j + 1] = a[1]; f[4 * j + 2] = b[0]; f[4 * j + 3] = b[1];
        }
    } else if constexpr (FMT == FP4_E2M1) {
        f32x2_t v;
        v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(lo, sf, 0); f[0] = v[0]; f[1] = v[1];
        v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(lo, sf, 1); f[2] = v[0]; f[3] = v[1];
        v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(lo, sf, 2); f[4] = v[0]; f[5] = v[1];
        v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(lo, sf, 3); f[6] = v[0]; f[7] = v[1];
    } else if constexpr (FMT == FP6_E3M2 || FMT == FP6_E2M3) {
        const u32x6_t_ d = {lo, hi, 0u, 0u, 0u, 0u};
        const f32x32_t v = FMT == FP6_E2M3 ? __builtin_amdgcn_cvt_scalef32_pk32_f32_fp6(d, sf)
                                           : __builtin_amdgcn_cvt_scalef32_pk32_f32_bf6(d, sf);
#pragma unroll
        for (int i = 0; i < 8; i++) f[i] = v[i];
    }
}

template <int DST>
__device__ __forceinline__ void store8(void *dst, int64_t at, const float (&f)[8], int n = 8)
{
    uint32_t h[4];   // hardware packed convert: round to nearest even, NaN stays NaN
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const f32x2_t pr = {f[2 * k], f[2 * k + 1]};
        h[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2_t_));
    }
    if (DST == DT_F32) {
        float *d = reinterpret_cast<float *>(dst) + at;
        if (n == 8) {
            *reinterpret_cast<float4 *>(d) = make_float4(f[0], f[1], f[2], f[3]);
            *reinterpret_cast<float4 *>(d + 4) = make_float4(f[4], f[5], f[6], f[7]);
        } else {
#pragma unroll
            for (int i = 0; i < 8; i++)
                if (i < n) d[i] = f[i];
        }
    } else {
        uint16_t *d = reinterpret_cast<uint16_t *>(dst) + at;
        if (n == 8) {
            st16(d, make_uint4(h[0], h[1], h[2], h[3]));
        } else {
#pragma unroll
            for (int i = 0; i < 8; i++)
                if (i < n) d[i] = (uint16_t)(h[i >> 1] >> (16 * (i & 1)));
        }
    }
}

// Blocks along the last axis: the tensor is one run of 8-code units (the fill of partial last blocks
// included).  FLAT, a dense result of whole blocks: unit u -> dst[8u .. 8u+7], no row arithmetic.
// Otherwise the rows of the result are those of `geom` and the fill is skipped.  A thread takes U
// units 256 apart and requests all of them (streaming loads) before it converts the first, so that a
// wave has U loads in flight; adjacent lanes write adjacent 16 (bf16) or 32 (Float32) bytes.
// U = 4 for one run.  Rows take one unit per thread and ordinary loads: the codes of such tensors are mostly in cache when they
// are read (119 x 202558 E5M2 -> Float32: U = 4 and streaming loads 34.6 us, U = 1 and streaming loads 31.4, this form
// 25.1; 4864 x 4960 in rows of 4968, INT8 -> bf16: 15.1, 15.0, 12.3).
constexpr int DQ_U = 4;
template <int FMT, int DST, bool FLAT, int U = FLAT ? DQ_U : 1>
__global__ __launch_bounds__(256) void dequant_row_kernel(const uint8_t *__restrict__ elems, const uint8_t *__restrict__ scales,
                                                          void *__restrict__ dst, int64_t n_units, RowGeom geom)
{
    constexpr int w = Fmt<FMT>::bits;
    const int64_t base = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
    uint32_t lo[U], hi[U], s[U];
#pragma unroll
    for (int i = 0; i < U; i++) {
        const int64_t u = base + i * 256;
        lo[i] = hi[i] = 0; s[i] = 127;
        if (u < n_units) {
            const uint8_t *p = elems + u * w;
            if (w == 8) { const uint2 d = FLAT ? ld8_nt(p) : *reinterpret_cast<const uint2 *>(p); lo[i] = d.x; hi[i] = d.y; }
            else if (w == 4) lo[i] = FLAT ? ld4_nt(p) : *reinterpret_cast<const uint32_t *>(p);
            else { lo[i] = ld2_nt(p) | (ld2_nt(p + 2) << 16); hi[i] = ld2_nt(p + 4); }
            s[i] = scales[u >> 2];
        }
    }
#pragma unroll
    for (int i = 0; i < U; i++) {
        const int64_t u = base + i * 256;
        if (u >= n_units) continue;
        float f[8];
        decode8_regs<FMT>(lo[i], hi[i], s[i], f);
        if (FLAT) {
            store8<DST>(dst, u * 8, f);
        } else {
            int n;
            const int64_t at = geom.at((uint32_t)u, 8, n);
            if (n > 0) store8<DST>(dst, at, f, n);
        }
    }
}

// The same for 8-bit codes and Float32 output with 4 codes per lane, so that every store instruction
// of a wave writes one gap-free kilobyte (with 8 codes per lane a lane's 32 bytes leave as two stores
// that each cover every other 16 bytes).
template <int FMT>
__global__ __launch_bounds__(256) void dequant_flat4_kernel(const uint8_t *__restrict__ elems, const uint8_t *__restrict__ scales,
                                                            float *__restrict__ dst, int64_t n_quads)
{
    static_assert(Fmt<FMT>::bits == 8, "one dword = four codes");
    const int64_t base = (int64_t)blockIdx.x * (256 * DQ_U) + threadIdx.x;
    uint32_t c[DQ_U], s[DQ_U];
#pragma unroll
    for (int i = 0; i < DQ_U; i++) {
        const int64_t u = base + i * 256;
        c[i] = 0; s[i] = 127;
        if (u < n_quads) { c[i] = ld4_nt(elems + u * 4); s[i] = scales[u >> 3]; }
    }
#pragma unroll
    for (int i = 0; i < DQ_U; i++) {
        const int64_t u = base + i * 256;
        if (u >= n_quads) continue;
        float4 v;
        if (FMT == INT8 || s[i] == SCALE_NAN) {
            v = make_float4(decode_scaled<FMT>(c[i] & 0xFFu, s[i]), decode_scaled<FMT>((c[i] >> 8) & 0xFFu, s[i]),
                            decode_scaled<FMT>((c[i] >> 16) & 0xFFu, s[i]), decode_scaled<FMT>(c[i] >> 24, s[i]));
        } else {
            const float sf = __uint_as_float(s[i] << 23);
            f32x2_t a, b;
            if (FMT == FP8_E4M3) {
                a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c[i], sf, false);
                b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(c[i], sf, true);
            } else {
                a = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(c[i], sf, false);
                b = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(c[i], sf, true);
            }
            v = make_float4(a[0], a[1], b[0], b[1]);
        }
        *reinterpret_cast<float4 *>(dst + u * 4) = v;
    }
}

// Axis 0 through LDS: the MX tensor is the cast of the transpose ([n_out][plen] with the block axis
// contiguous, plen = len rounded up to whole blocks), the result is row-major [len][n_out].  A work-group
// takes 64 lines x 128 positions: 16 lanes read one line's 128 codes side by side (coalesced), every
// lane decodes 8 of them, the values go transposed into a [128][64] Float32 tile (pitch 65: reads below
// are conflict-free, writes two-way), and the tile leaves row by row with 16-byte stores, adjacent lanes
// writing adjacent 16 bytes, so that every store instruction fills whole 128-byte lines (a lane that
// owns a longer run and stores it 16 bytes at a time leaves every line to several instructions, which
// measured 60 instead of 40 us).  Whole tiles take the form without bounds checks; blockIdx.z walks a
// batch of tensors (128 tensors of 2048 x 128 bf16 <-> E4M3: cast and dequantize took 949 us with a launch
// per tensor, 42 us with one each, 4.0 TB/s).
constexpr int DQT_O = 64, DQT_L = 128, DQT_PITCH = 65;
template <int FMT, int DST, bool WHOLE>
__global__ __launch_bounds__(256) void dequant_tr_tile_kernel(const uint8_t *__restrict__ elems,
                                                              const uint8_t *__restrict__ scales, void *__restrict__ dst,
                                                              int64_t n_out, int64_t len, int64_t ld, Batch batch)
{
    constexpr int w = Fmt<FMT>::bits;
    __shared__ float tile[DQT_L * DQT_PITCH];
    elems += blockIdx.z * batch.elems;
    scales += blockIdx.z * batch.scales;
    dst = static_cast<char *>(dst) + blockIdx.z * batch.src * (DST == DT_F32 ? 4 : 2);
    const int t = threadIdx.x;
    const int64_t tiles_o = (n_out + DQT_O - 1) / DQT_O;
    const int64_t O0 = (int64_t)(blockIdx.x % tiles_o) * DQT_O, L0 = (int64_t)(blockIdx.x / tiles_o) * DQT_L;
    const int64_t units_per_row = (len + BLOCK - 1) / BLOCK * (BLOCK / 8);
#pragma unroll
    for (int p = 0; p < 4; p++) {
        const int o = 16 * p + (t >> 4), u = t & 15;
        float f[8];
        if (WHOLE || (O0 + o < n_out && L0 / 8 + u < units_per_row)) {
            const int64_t unit = (O0 + o) * units_per_row + L0 / 8 + u;
            const uint32_t s = scales[unit / 4];
            if (FMT != INT8 && s != SCALE_NAN) {
                decode8_hw<FMT>(elems + unit * w, s, f);
            } else {
                uint32_t c[8];
                load_codes8<FMT>(elems + unit * w, c);
#pragma unroll
                for (int i = 0; i < 8; i++) f[i] = decode_scaled<FMT>(c[i], s);
            }
#pragma unroll
            for (int i = 0; i < 8; i++) tile[(8 * u + i) * DQT_PITCH + o] = f[i];
        }
    }
    __syncthreads();
    // a result row of the tile is 64 values = 16 lanes x 16 bytes (Float32, 16 rows per pass) or 8 lanes
    // (bf16, 32 rows per pass)
    constexpr int PER = DST == DT_F32 ? 4 : 8, LPR = DQT_O / PER, RPP = 256 / LPR;
    const int q = t % LPR;
    const int64_t left = WHOLE ? PER : n_out - O0 - PER * q;
    const int n = left >= PER ? PER : left > 0 ? (int)left : 0;
#pragma unroll
    for (int p = 0; p < DQT_L / RPP; p++) {
        const int row = RPP * p + t / LPR;
        if (!WHOLE && L0 + row >= len) break;
        const float *src = tile + row * DQT_PITCH + PER * q;
        const int64_t at = (L0 + row) * ld + O0 + PER * q;
        if constexpr (DST == DT_F32) {
            float *d = reinterpret_cast<float *>(dst) + at;
            if (WHOLE || n == 4) {
                *reinterpret_cast<float4 *>(d) = make_float4(src[0], src[1], src[2], src[3]);
            } else {
                for (int i = 0; i < n; i++) d[i] = src[i];
            }
        } else {
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; j++) f[j] = (WHOLE || j < n) ? src[j] : 0.f;
            if (WHOLE || n == 8) store8<DST>(dst, at, f);
            else if (n > 0) store8<DST>(dst, at, f, n);
        }
    }
}

// Axis 0 without LDS: one lane per 8 codes of a line; adjacent lanes take adjacent lines, so that the stores of a wave coalesce
// across it (2 or 4 bytes each).  Ahead of the tile kernel where a tile would be mostly empty or the tensor is small (see launch_t).
template <int FMT, int DST>
__global__ __launch_bounds__(256) void dequant_tr_kernel(const uint8_t *__restrict__ elems, const uint8_t *__restrict__ scales,
                                                         void *__restrict__ dst, FastDiv n_out, int64_t len, int64_t ld,
                                                         uint32_t n_units, Batch batch)
{
    constexpr int w = Fmt<FMT>::bits;
    elems += blockIdx.z * batch.elems;
    scales += blockIdx.z * batch.scales;
    dst = static_cast<char *>(dst) + blockIdx.z * batch.src * (DST == DT_F32 ? 4 : 2);
    const uint32_t u = blockIdx.x * 256 + threadIdx.x;
    if (u >= n_units) return;
    const uint32_t q = n_out(u), o = u - q * n_out.d;
    const int64_t unit = o * ((len + BLOCK - 1) / BLOCK * (BLOCK / 8)) + q, l = (int64_t)q * 8;
    const uint32_t s = scales[unit / 4];
    float f[8];
    if (FMT != INT8 && s != SCALE_NAN) {
        decode8_hw<FMT>(elems + unit * w, s, f);
    } else {
        uint32_t c[8];
        load_codes8<FMT>(elems + unit * w, c);
#pragma unroll
        for (int i = 0; i < 8; i++) f[i] = decode_scaled<FMT>(c[i], s);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
        if (l + i >= len) break;
        if (DST == DT_F32) reinterpret_cast<float *>(dst)[(l + i) * ld + o] = f[i];
        else reinterpret_cast<uint16_t *>(dst)[(l + i) * ld + o] = (uint16_t)f32_to_bf16_bits(f[i]);
    }
}

// Which tensors of remainders go through the tile kernel (whole tiles always do, and what the other cannot number in 31 bits): both
// dimensions fill most of a tile and there are enough of them.  Without LDS / tiles, us, Float32: 31 x 270600 E4M3 10.6 / 16.9,
// 90 x 93200 E3M2 9.0 / 12.0, 200 x 41944 E4M3 15.1 / 11.6; lines of few columns, 699057 x 12 E4M3 10 / 16, 174759 x 48 11 / 10.6,
// 86487 x 97 16 / 13; and 2^21 elements, 257 x 8160 4.3 / 4.7.  A second tile that is nearly empty, 130 x 129048: E2M1 15.5 / 21.9, E3M2
// 18.8 / 23.2, but 129 x 65024 E4M3 21 / 12.6 (a line of whole 128-byte lines of codes and a bit suits the reads without LDS badly).
static bool tr_tiles_pay(int64_t n, int64_t rows, int64_t cols, int w)
{
    const int64_t lines = (rows + DQT_L - 1) / DQT_L * DQT_L;
    if (cols % DQT_O == 0 && rows % DQT_L == 0) return true;
    if (cols * ((rows + 7) / 8) > 0x7FFFFFFF) return true;
    return rows >= DQT_L && cols >= 96 && n * rows * cols >= ((int64_t)1 << 22) && (w == 8 || rows * 5 >= lines * 3);
}

template <int FMT, int DST>
static hipError_t launch_t(const uint8_t *elems, const uint8_t *scales, int64_t rows, int64_t cols, int axis, void *dst,
                           int64_t ld, hipStream_t st, const Batch &batch)
{
    constexpr int w = Fmt<FMT>::bits;
    constexpr int64_t esz = DST == DT_F32 ? 4 : 2;
    if (axis == 0) {
        const int64_t tiles = ((cols + DQT_O - 1) / DQT_O) * ((rows + DQT_L - 1) / DQT_L);
        const bool tiled = tr_tiles_pay(batch.n, rows, cols, w);
        if (tiled && tiles > 0x7FFFFFFF) return hipErrorNotSupported;
        const int64_t n_units = cols * ((rows + 7) / 8);
        for (int64_t i = 0; i < batch.n; i += 65535) {
            const dim3 grid((unsigned)(tiled ? tiles : (n_units + 255) / 256), 1,
                            (unsigned)(batch.n - i < 65535 ? batch.n - i : 65535));
            const uint8_t *e = elems + i * batch.elems, *sc = scales + i * batch.scales;
            void *d = static_cast<char *>(dst) + i * batch.src * esz;
            if (!tiled)
                hipLaunchKernelGGL((dequant_tr_kernel<FMT, DST>), grid, dim3(256), 0, st, e, sc, d, fast_div(cols), rows, ld,
                                   (uint32_t)n_units, batch);
            else if (cols % DQT_O == 0 && rows % DQT_L == 0)
                hipLaunchKernelGGL((dequant_tr_tile_kernel<FMT, DST, true>), grid, dim3(256), 0, st, e, sc, d, cols, rows, ld, batch);
            else
                hipLaunchKernelGGL((dequant_tr_tile_kernel<FMT, DST, false>), grid, dim3(256), 0, st, e, sc, d, cols, rows, ld, batch);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    // axis 1: the MX tensor is one run of batch.n * rows lines (a batch has dense inputs)
    const int64_t upr = (cols + BLOCK - 1) / BLOCK * (BLOCK / 8), n_units = batch.n * rows * upr;
    if (ld == cols && cols % BLOCK == 0 && (batch.n == 1 || batch.src == rows * ld)) {
        if constexpr (DST == DT_F32 && w == 8) {
            const int64_t nq = n_units * 2, nbq = (nq + 256 * DQ_U - 1) / (256 * DQ_U);
            if (nbq <= 0x7FFFFFFF) {
                hipLaunchKernelGGL((dequant_flat4_kernel<FMT>), dim3((unsigned)nbq), dim3(256), 0, st, elems, scales,
                                   static_cast<float *>(dst), nq);
                return hipGetLastError();
            }
        }
        const int64_t nb = (n_units + 256 * DQ_U - 1) / (256 * DQ_U);
        if (nb <= 0x7FFFFFFF) {
            hipLaunchKernelGGL((dequant_row_kernel<FMT, DST, true>), dim3((unsigned)nb), dim3(256), 0, st, elems, scales, dst, n_units,
                               RowGeom{});
            return hipGetLastError();
        }
    }
    // strided or ragged rows: units are numbered in 31 bits, so very large tensors go a run of rows at a time
    const int64_t most = 0x7FFFFFFF / upr;
    if (most < 1) return hipErrorNotSupported;
    const bool once = batch.n * rows <= most;
    for (int64_t i = 0; i < (once ? 1 : batch.n); i++)
        for (int64_t r = 0; r < rows; r += once ? rows : most) {
            const int64_t nr = once || rows - r < most ? rows - r : most, nz = once ? batch.n : 1, line = i * rows + r, n = nz * nr * upr;
            hipLaunchKernelGGL((dequant_row_kernel<FMT, DST, false>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                               elems + line * upr * w, scales + line * (upr / 4), static_cast<char *>(dst) + (i * batch.src + r * ld) * esz, n,
                               row_geom(nz, nr, cols, ld, nz > 1 ? batch.src : nr * ld, 8));
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
    return hipSuccess;
}

template <int DST>
static hipError_t launch_f(int fmt, const uint8_t *elems, const uint8_t *scales, int64_t rows, int64_t cols, int axis,
                           void *dst, int64_t ld, hipStream_t st, const Batch &batch)
{
    switch (fmt) {
        case FP8_E4M3: return launch_t<FP8_E4M3, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
        case FP8_E5M2: return launch_t<FP8_E5M2, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
        case FP6_E3M2: return launch_t<FP6_E3M2, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
        case FP6_E2M3: return launch_t<FP6_E2M3, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
        case FP4_E2M1: return launch_t<FP4_E2M1, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
        default:       return launch_t<INT8, DST>(elems, scales, rows, cols, axis, dst, ld, st, batch);
    }
}

hipError_t launch_dequant(const uint8_t *elems, const uint8_t *scales, int fmt, int64_t rows, int64_t cols, int axis,
                          void *dst, int dst_dt, int64_t ld, hipStream_t st, const Batch &batch)
{
    return dst_dt == DT_F32 ? launch_f<DT_F32>(fmt, elems, scales, rows, cols, axis, dst, ld, st, batch)
                            : launch_f<DT_BF16>(fmt, elems, scales, rows, cols, axis, dst, ld, st, batch);
}

}  // namespace mx
