// MXINT8 x MXINT8 GEMM (Section 4.1 of arXiv 2310.10537; MXINT8 is the format of Table 1
// with two's-complement elements and an implied scale of 2^-6).  The block-scaled matrix
// instruction has no integer form, so each 32-element block is one plain
// V_MFMA_I32_32X32X32_I8 -- its 32 products and their sum are exact integers -- and
// the block's contribution X_A * X_B * sum is added in Float32 with an exact
// power-of-two scaling (a Float32 factor where the scales allow it, ldexp otherwise):
//   C[m][n] += float(sum_j qa[m][32b+j] * qb[n][32b+j]) * 2^(sA[m][b] + sB[n][b] - 254 - 12).
// Operand layout of the instruction (the same as each 32-wide half of the 8-bit f8f6f4 form):
// lane l holds, for row / column l % 32, the 16 consecutive K bytes [16 * (l / 32), + 16);
// result register t of lane l is C[8*(t/4) + 4*(l/32) + t%4][l % 32].
// One wave per 32 x 32 output tile, operands straight from global memory, any shape.  The
// A scale of a block is needed per output row, i.e. per result register: the 32 row bytes
// go through a wave-private LDS line and come back as the sixteen dwords a lane needs.
//
// Larger products take a faster, equally exact route: an element times its block's scale, q 2^(s - 133), is a bf16 number (q has
// eight significant bits at most), the product of two such numbers is exact in Float32, and so C is the plain bf16 product of the
// scaled elements on the bf16 matrix instruction (mx_gemm_bf16.hip), Float32 sums as everywhere.  That holds while no sum can leave
// the range of Float32; int8_widen_kernel notes the largest scales, and the direct kernel's tiles -- launched after the product, left at
// once as a rule -- recompute the parts of C where it does not.  (The 8-bit integer
// instruction is twice as fast as the bf16 one, but every block's sums have to be scaled by the vector pipe: 48 instructions for
// 32 clocks of it.  Splitting q into two E2M3 halves, four products on the block-scaled instruction at four times the bf16 rate, moves
// three bytes an element instead of two for the same matrix work: 8192 x 4096 x 4096 388 us where this takes 227.)
#include "mx_device.hpp"
#include "mx_launch.hpp"

namespace mx {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v16i_t __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void wave_lds_sync8()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
}

// Adds one block's contribution to the 16 accumulators of a lane: acc[t] += p[t] * 2^(sA[row t] + sB - 266).
// sa / sb are the scale bytes of the lane's own row / column (lane i = row i and column i of the tile);
// the per-row bytes travel through the wave's 32-dword LDS line.  When every scale byte of the block is
// within [70, 196] (or the NaN byte) the two factors 2^(s - 133) and their product are normal Float32
// numbers (exponent sum in [-126, 126]), so is every scaled sum: one multiply and one fused
// multiply-add per entry, the row factor arriving ready-made.  Any other scale byte in the wave's block
// sends the whole wave through the exact power-of-two scaling of ldexp (3 more instructions per entry).
__device__ __forceinline__ uint32_t i8_factor_bits(uint32_t s) { return s == SCALE_NAN ? 0x7FC00000u : (s - 6u) << 23; }
__device__ __forceinline__ bool i8_factor_ok(uint32_t s) { return s - 70u <= 126u || s == SCALE_NAN; }

__device__ __forceinline__ void i8_accumulate(float (&acc)[16], const v16i_t &p, uint32_t sa, uint32_t sb, uint32_t *line,
                                              int i, int g)
{
    const bool plain = i8_factor_ok(sa) && i8_factor_ok(sb);
    const bool fast = __builtin_amdgcn_ballot_w64(!plain) == 0;   // uniform over the wave
    if (g == 0) line[i] = fast ? i8_factor_bits(sa) : sa;
    wave_lds_sync8();
    uint32_t w[16];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint4 r = *reinterpret_cast<const uint4 *>(line + 8 * q + 4 * g);   // rows 8q + 4g .. + 3 = registers 4q .. 4q + 3
        w[4 * q] = r.x; w[4 * q + 1] = r.y; w[4 * q + 2] = r.z; w[4 * q + 3] = r.w;
    }
    if (fast) {
        const float fb = __uint_as_float(i8_factor_bits(sb));
#pragma unroll
        for (int t = 0; t < 16; t++) acc[t] = fmaf((float)p[t], __uint_as_float(w[t]) * fb, acc[t]);
    } else {
#pragma unroll
        for (int t = 0; t < 16; t++) {
            float term = ldexpf((float)p[t], (int)w[t] + (int)sb - 254 - 12);
            if (w[t] == SCALE_NAN || sb == SCALE_NAN) term = __uint_as_float(0x7FC00000u);
            acc[t] += term;
        }
    }
    wave_lds_sync8();   // the line is rewritten for the next block
}

// ---------------------------------------------------------------------------------------------
// MXINT8 -> bf16.  A block's elements times its scale are q 2^(s - 133), |q| <= 128: exact in bf16, which holds eight significant
// bits down to 2^-126 and whole multiples of 2^-133 below (the matrix instruction takes and returns such numbers as they are).  Only
// -128 2^(254 - 133) = -2^128 has no bf16 value; a NaN scale makes its block's values NaN.  Products and sums below 2^-126 are as exact
// as Float32 is there.  At the other end a sum of K products must stay finite whatever its signs, as a block's sum does in
// integers: |product| <= 2^(sA + sB - 252), so sA + sB + log2 K <= 379.  Each work-group leaves the largest scale byte of its elements
// other than zero in a word of its own (OUT_OF_RANGE: a value without a bf16 form); gemm_int8_repair_kernel, launched behind the product on
// few work-groups, looks at all of them and recomputes the 64 x 64 tiles whose rows and columns do not fit together.
// Bound by memory: 3 bytes an element, 16-byte stores.
// ---------------------------------------------------------------------------------------------
constexpr int WIDEN_PER = 4;                                   // pieces of eight elements per lane
constexpr int WIDEN_ELEMS = 256 * 8 * WIDEN_PER;               // elements per work-group
constexpr uint32_t OUT_OF_RANGE = 1000;

// the largest of the work-group's (256 threads) values, for all of them
__device__ __forceinline__ uint32_t group_max(uint32_t m, uint32_t *part)
{
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = (uint32_t)__shfl_xor((int)m, o);
        m = m > t ? m : t;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; k++) m = m > part[k] ? m : part[k];
    return m;
}

__global__ __launch_bounds__(256) void int8_widen_kernel(const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As, int64_t a_elems,
                                                         const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs, int64_t b_elems,
                                                         uint16_t *__restrict__ Aw, uint16_t *__restrict__ Bw, uint32_t *__restrict__ range,
                                                         unsigned a_groups)
{
    __shared__ uint32_t part[4];
    const bool isb = blockIdx.x >= a_groups;
    const uint8_t *e = isb ? Be : Ae, *sc = isb ? Bs : As;
    uint16_t *w = isb ? Bw : Aw;
    const int64_t n = isb ? b_elems : a_elems, base = (int64_t)(blockIdx.x - (isb ? a_groups : 0)) * WIDEN_ELEMS + threadIdx.x * 8;
    uint2 q[WIDEN_PER];
    uint32_t s[WIDEN_PER];
#pragma unroll
    for (int k = 0; k < WIDEN_PER; k++) {
        const int64_t at = base + k * 2048;
        q[k] = make_uint2(0, 0);
        s[k] = 127;
        if (at < n) {
            q[k] = *reinterpret_cast<const uint2 *>(e + at);
            s[k] = sc[at >> 5];
        }
    }
    uint32_t hi = 0;
#pragma unroll
    for (int k = 0; k < WIDEN_PER; k++) {
        const float f = __uint_as_float(s[k] == SCALE_NAN ? 0x7FC00000u : s[k] >= 7 ? (s[k] - 6u) << 23 : 0x00400000u >> (6u - s[k]));
        uint32_t d[4], most = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int dw = (int)(i < 2 ? q[k].x : q[k].y), sh = 16 * (i & 1);
            const uint32_t v0 = __float_as_uint((float)((dw << (24 - sh)) >> 24) * f), v1 = __float_as_uint((float)((dw << (16 - sh)) >> 24) * f);
            d[i] = __builtin_amdgcn_perm(v1, v0, 0x07060302);
            most = most > v0 ? most : v0;
            most = most > v1 ? most : v1;
        }
        // (-2^128 is -Inf, the largest of all values but NaN by their bits)
        const uint32_t top = s[k] == SCALE_NAN ? 0 : most == 0xFF800000u ? OUT_OF_RANGE : (q[k].x | q[k].y) != 0 ? s[k] : 0;
        hi = hi > top ? hi : top;
        const int64_t at = base + k * 2048;
        if (at < n) st16(reinterpret_cast<uint8_t *>(w + at), make_uint4(d[0], d[1], d[2], d[3]));
    }
    hi = group_max(hi, part);
    if (threadIdx.x == 0) range[blockIdx.x] = hi;
}

// The largest of the words [first, last] of what int8_widen_kernel left, for every thread of the work-group (256).  Bound by the
// latency of its loads: eight in flight, where one after the other took 16.9 us over the 6144 words of 8192 x 4096 x 4096 (4.6 us so).
__device__ __forceinline__ uint32_t largest_scale(const uint32_t *__restrict__ range, unsigned first, unsigned last, uint32_t *part)
{
    constexpr unsigned AHEAD = 8;
    uint32_t m = 0;
    for (unsigned k0 = first + threadIdx.x; k0 <= last; k0 += AHEAD * 256) {
        uint32_t r[AHEAD];
#pragma unroll
        for (unsigned j = 0; j < AHEAD; j++) r[j] = range[k0 + j * 256 <= last ? k0 + j * 256 : last];    // (beyond the end: the last word again)
#pragma unroll
        for (unsigned j = 0; j < AHEAD; j++) m = m > r[j] ? m : r[j];
    }
    return group_max(m, part);
}

// One tile of 64 x 64
template <int CDT>
__device__ __forceinline__ void int8_tile(int64_t M, int64_t N, int64_t K, const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                          const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs, void *__restrict__ C, int64_t ldc,
                                          int64_t tile_m, int64_t tile_n, uint32_t *lds_all)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t *lds = lds_all + wave * 32;
    const int64_t m0 = tile_m * 64 + (wave >> 1) * 32;
    const int64_t n0 = tile_n * 64 + (wave & 1) * 32;
    const int i = lane & 31, g = lane >> 5;
    const int64_t nkb = K / BLOCK;
    const int64_t row = m0 + i, col = n0 + i;
    const bool rv = row < M, cv = col < N;
    const int64_t rowc = rv ? row : 0, colc = cv ? col : 0;   // keep addresses in range for masked lanes

    float acc[16];
#pragma unroll
    for (int t = 0; t < 16; t++) acc[t] = 0.f;

    for (int64_t kb = 0; kb < nkb; kb++) {
        const uint4 qa = ld16(Ae + rowc * K + kb * BLOCK + 16 * g);
        const uint4 qb = ld16(Be + colc * K + kb * BLOCK + 16 * g);
        const uint32_t sa = As[rowc * nkb + kb], sb = Bs[colc * nkb + kb];
        const v4i_t a = rv ? v4i_t{(int)qa.x, (int)qa.y, (int)qa.z, (int)qa.w} : v4i_t{0, 0, 0, 0};
        const v4i_t b = cv ? v4i_t{(int)qb.x, (int)qb.y, (int)qb.z, (int)qb.w} : v4i_t{0, 0, 0, 0};
        v16i_t z;
#pragma unroll
        for (int t = 0; t < 16; t++) z[t] = 0;
        const v16i_t p = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, z, 0, 0, 0);
        i8_accumulate(acc, p, sa, sb, lds, i, g);
    }

#pragma unroll
    for (int t = 0; t < 16; t++) {
        const int64_t r = m0 + 8 * (t / 4) + 4 * g + (t % 4);
        if (r < M && cv) {
            if (CDT == DT_F32) reinterpret_cast<float *>(C)[r * ldc + col] = acc[t];
            else reinterpret_cast<uint16_t *>(C)[r * ldc + col] = (uint16_t)f32_to_bf16_bits(acc[t]);
        }
    }
}

template <int CDT>
__global__ __launch_bounds__(256) void gemm_int8_kernel(int64_t M, int64_t N, int64_t K, const uint8_t *__restrict__ Ae,
                                                        const uint8_t *__restrict__ As, const uint8_t *__restrict__ Be,
                                                        const uint8_t *__restrict__ Bs, void *__restrict__ C, int64_t ldc)
{
    __shared__ __attribute__((aligned(16))) uint32_t lds_all[4 * 32];
    int8_tile<CDT>(M, N, K, Ae, As, Be, Bs, C, ldc, blockIdx.y, blockIdx.x, lds_all);
}

// Behind the product of the bf16 values, on few work-groups: nothing to repair, as a rule.  limit: the largest sum of two scale bytes
// that the product allows.  A tile's words are those of the work-groups that widened its rows or columns, neighbours among them.
template <int CDT>
__global__ __launch_bounds__(256) void gemm_int8_repair_kernel(int64_t M, int64_t N, int64_t K, const uint8_t *__restrict__ Ae,
                                                               const uint8_t *__restrict__ As, const uint8_t *__restrict__ Be,
                                                               const uint8_t *__restrict__ Bs, void *__restrict__ C, int64_t ldc,
                                                               const uint32_t *__restrict__ range, unsigned n_a, unsigned n_b, unsigned limit)
{
    __shared__ uint32_t part[4];
    if (largest_scale(range, 0, n_a - 1, part) + largest_scale(range + n_a, 0, n_b - 1, part) <= limit) return;
    __shared__ __attribute__((aligned(16))) uint32_t lds_all[4 * 32];
    const int64_t tiles_n = (N + 63) / 64, tiles = tiles_n * ((M + 63) / 64);
    auto strip = [&](const uint32_t *words, int64_t t, int64_t rows) {
        const int64_t end = 64 * t + 64 < rows ? 64 * t + 64 : rows;
        return largest_scale(words, (unsigned)(64 * t * K / WIDEN_ELEMS), (unsigned)((end * K - 1) / WIDEN_ELEMS), part);
    };
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t tm = tile / tiles_n, tn = tile % tiles_n;
        if (strip(range, tm, M) + strip(range + n_a, tn, N) > limit) int8_tile<CDT>(M, N, K, Ae, As, Be, Bs, C, ldc, tm, tn, lds_all);
    }
}

// Few rows of A (a decoding step): the kernel above gives such a problem N / 32 waves that each walk
// the whole K range alone, one load-then-multiply after the other.  Here eight waves share 32 rows
// x 32 columns of C, each a contiguous eighth of the blocks, with the operands of four blocks
// requested before the first is multiplied; the eight partial sums meet in LDS and are added in
// the order w0 + w1 + ... + w7.
constexpr int I8_WAVES = 8, I8_U = 4;
template <int CDT>
__global__ __launch_bounds__(64 * I8_WAVES) void gemm_int8_shared_k_kernel(int64_t M, int64_t N, int64_t K,
                                                                            const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                                                            const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                                            void *__restrict__ C, int64_t ldc)
{
    __shared__ __attribute__((aligned(16))) uint32_t lds_all[I8_WAVES * 32];
    __shared__ float red[I8_WAVES - 1][16][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t *lds = lds_all + wave * 32;
    const int64_t m0 = (int64_t)blockIdx.y * 32, n0 = (int64_t)blockIdx.x * 32;
    const int i = lane & 31, g = lane >> 5;
    const int64_t nkb = K / BLOCK;
    const int64_t chunk = (nkb + I8_WAVES - 1) / I8_WAVES;
    const int64_t kb_begin = wave * chunk, kb_end = kb_begin + chunk < nkb ? kb_begin + chunk : nkb;
    const int64_t row = m0 + i, col = n0 + i;
    const bool rv = row < M, cv = col < N;
    const int64_t rowc = rv ? row : 0, colc = cv ? col : 0;   // keep addresses in range for masked lanes

    float acc[16];
#pragma unroll
    for (int t = 0; t < 16; t++) acc[t] = 0.f;

    for (int64_t kb0 = kb_begin; kb0 < kb_end; kb0 += I8_U) {
        uint4 qa[I8_U], qb[I8_U];
        uint32_t sa[I8_U], sb[I8_U];
#pragma unroll
        for (int u = 0; u < I8_U; u++) {
            const int64_t kb = kb0 + u < kb_end ? kb0 + u : kb_end - 1;   // past the slice: a valid block, result unused
            qa[u] = ld16(Ae + rowc * K + kb * BLOCK + 16 * g);
            qb[u] = ld16(Be + colc * K + kb * BLOCK + 16 * g);
            sa[u] = As[rowc * nkb + kb];
            sb[u] = Bs[colc * nkb + kb];
        }
#pragma unroll
        for (int u = 0; u < I8_U; u++) {
            if (kb0 + u >= kb_end) break;                                 // wave-uniform
            const v4i_t a = rv ? v4i_t{(int)qa[u].x, (int)qa[u].y, (int)qa[u].z, (int)qa[u].w} : v4i_t{0, 0, 0, 0};
            const v4i_t b = cv ? v4i_t{(int)qb[u].x, (int)qb[u].y, (int)qb[u].z, (int)qb[u].w} : v4i_t{0, 0, 0, 0};
            v16i_t z;
#pragma unroll
            for (int t = 0; t < 16; t++) z[t] = 0;
            const v16i_t p = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, z, 0, 0, 0);
            i8_accumulate(acc, p, sa[u], sb[u], lds, i, g);
        }
    }

    if (wave > 0) {
#pragma unroll
        for (int t = 0; t < 16; t++) red[wave - 1][t][lane] = acc[t];
    }
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int t = 0; t < 16; t++) {
        float v = acc[t];
#pragma unroll
        for (int w = 0; w < I8_WAVES - 1; w++) v += red[w][t][lane];
        const int64_t r = m0 + 8 * (t / 4) + 4 * g + (t % 4);
        if (r < M && cv) {
            if (CDT == DT_F32) reinterpret_cast<float *>(C)[r * ldc + col] = v;
            else reinterpret_cast<uint16_t *>(C)[r * ldc + col] = (uint16_t)f32_to_bf16_bits(v);
        }
    }
}

// The same with the operands staged through LDS (K a multiple of 128).  Above, every lane of an operand
// load addresses a different matrix row, so one load instruction touches 64 cache lines and uses 16 bytes
// of each; here a wave fetches 128 bytes of each row at a time with loads whose adjacent lanes read
// adjacent 16 bytes (every line touched once), parks the pieces in a private LDS tile -- rows of 128
// bytes, 16-byte piece c of row r in slot c ^ ((r / 2) % 8), which keeps both the parking stores and the
// operand reads free of bank conflicts -- and multiplies its four blocks from there while the next 128
// bytes are in flight.  MT tiles of 32 rows share the B tile of the work-group's 32 columns.  Rows beyond
// M and columns beyond N read the last valid one instead: their results are never stored.
// QN: groups of 8 rows of a tile that are scaled and stored (result registers 4q .. 4q + 3 are rows
// 8q + 4g .. + 3); a decoding step of at most 8 or 16 rows skips the rest.
template <int MT, int QN, int CDT>
__global__ __launch_bounds__(64 * I8_WAVES) void gemm_int8_lds_kernel(int64_t M, int64_t N, int64_t K,
                                                                       const uint8_t *__restrict__ Ae, const uint8_t *__restrict__ As,
                                                                       const uint8_t *__restrict__ Be, const uint8_t *__restrict__ Bs,
                                                                       void *__restrict__ C, int64_t ldc)
{
    constexpr int T_BYTES = 32 * 128, W_BYTES = (MT + 1) * T_BYTES;
    constexpr int RED_BYTES = (I8_WAVES - 1) * MT * 16 * 64 * 4;
    static_assert(I8_WAVES * W_BYTES >= RED_BYTES, "the partial sums reuse the staging tiles");
    __shared__ __attribute__((aligned(16))) uint8_t lds[I8_WAVES * W_BYTES];
    __shared__ __attribute__((aligned(16))) uint32_t lines[I8_WAVES * MT * 4 * 32];   // per wave, tile and block: 32 row words
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 31, g = lane >> 5;
    const int64_t n0 = (int64_t)blockIdx.x * 32, m0 = (int64_t)blockIdx.y * (32 * MT);
    const int64_t nkb = K / BLOCK, chunks = K / 128;
    const int64_t per_wave = (chunks + I8_WAVES - 1) / I8_WAVES;
    const int64_t c_begin = wave * per_wave, c_end = c_begin + per_wave < chunks ? c_begin + per_wave : chunks;
    uint8_t *tA = lds + wave * W_BYTES, *tB = tA + MT * T_BYTES;
    uint32_t *line = lines + wave * (MT * 4 * 32);

    const int lr = lane >> 3, lp = lane & 7;            // a wave-wide load: 8 rows x eight 16-byte pieces
    auto slot = [](int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); };
    auto clampi = [](int64_t v, int64_t hi) { return v < hi ? v : hi; };
    uint4 ra[MT][4], rb[4];
    uint32_t sa_d[MT], sb_d;
    auto request = [&](int64_t c) {
#pragma unroll
        for (int x = 0; x < MT; x++)
#pragma unroll
            for (int j = 0; j < 4; j++) ra[x][j] = ld16(Ae + clampi(m0 + 32 * x + 8 * j + lr, M - 1) * K + c * 128 + lp * 16);
#pragma unroll
        for (int j = 0; j < 4; j++) rb[j] = ld16(Be + clampi(n0 + 8 * j + lr, N - 1) * K + c * 128 + lp * 16);
#pragma unroll
        for (int x = 0; x < MT; x++) sa_d[x] = *reinterpret_cast<const uint32_t *>(As + clampi(m0 + 32 * x + i, M - 1) * nkb + c * 4);
        sb_d = *reinterpret_cast<const uint32_t *>(Bs + clampi(n0 + i, N - 1) * nkb + c * 4);
    };

    float acc[MT][16];
#pragma unroll
    for (int x = 0; x < MT; x++)
#pragma unroll
        for (int t = 0; t < 16; t++) acc[x][t] = 0.f;

    if (c_begin < c_end) request(c_begin);
    for (int64_t c = c_begin; c < c_end; c++) {
#pragma unroll
        for (int x = 0; x < MT; x++)
#pragma unroll
            for (int j = 0; j < 4; j++) *reinterpret_cast<uint4 *>(tA + x * T_BYTES + slot(8 * j + lr, lp)) = ra[x][j];
#pragma unroll
        for (int j = 0; j < 4; j++) *reinterpret_cast<uint4 *>(tB + slot(8 * j + lr, lp)) = rb[j];
        // The four scale bytes of row i (one per block of the chunk) go to the wave's lines next to the
        // operands, under the same wait: as ready-made Float32 factors when every scale byte of the chunk,
        // rows and columns, allows it (see i8_accumulate), as plain bytes otherwise.  The lower half-wave
        // writes blocks 0 and 1, the upper one blocks 2 and 3 (both hold row i's dword).
        uint32_t sa_c[MT];
#pragma unroll
        for (int x = 0; x < MT; x++) sa_c[x] = sa_d[x];
        const uint32_t sb_c = sb_d;
        bool plain = true;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            plain = plain && i8_factor_ok((sb_c >> (8 * b)) & 0xFFu);
#pragma unroll
            for (int x = 0; x < MT; x++) plain = plain && i8_factor_ok((sa_c[x] >> (8 * b)) & 0xFFu);
        }
        const bool fast = __builtin_amdgcn_ballot_w64(!plain) == 0;   // uniform over the wave
#pragma unroll
        for (int x = 0; x < MT; x++)
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int b = 2 * g + h;
                const uint32_t sbyte = (sa_c[x] >> (8 * b)) & 0xFFu;
                line[(x * 4 + b) * 32 + i] = fast ? i8_factor_bits(sbyte) : sbyte;
            }
        wave_lds_sync8();
        if (c + 1 < c_end) request(c + 1);
#pragma unroll
        for (int b = 0; b < 4; b++) {
            // lane (i, g) of the instruction: bytes [16 g, 16 g + 16) of block b of row / column i
            const uint4 qb = *reinterpret_cast<const uint4 *>(tB + slot(i, 2 * b + g));
            const v4i_t bv = {(int)qb.x, (int)qb.y, (int)qb.z, (int)qb.w};
            const uint32_t sbb = (sb_c >> (8 * b)) & 0xFFu;
            const float fb = __uint_as_float(i8_factor_bits(sbb));
#pragma unroll
            for (int x = 0; x < MT; x++) {
                const uint4 qa = *reinterpret_cast<const uint4 *>(tA + x * T_BYTES + slot(i, 2 * b + g));
                const v4i_t av = {(int)qa.x, (int)qa.y, (int)qa.z, (int)qa.w};
                uint32_t w[4 * QN];
#pragma unroll
                for (int q = 0; q < QN; q++) {
                    const uint4 r = *reinterpret_cast<const uint4 *>(line + (x * 4 + b) * 32 + 8 * q + 4 * g);   // rows 8q + 4g .. + 3
                    w[4 * q] = r.x; w[4 * q + 1] = r.y; w[4 * q + 2] = r.z; w[4 * q + 3] = r.w;
                }
                v16i_t z;
#pragma unroll
                for (int t = 0; t < 16; t++) z[t] = 0;
                const v16i_t p = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, z, 0, 0, 0);
                if (fast) {
#pragma unroll
                    for (int t = 0; t < 4 * QN; t++) acc[x][t] = fmaf((float)p[t], __uint_as_float(w[t]) * fb, acc[x][t]);
                } else {
#pragma unroll
                    for (int t = 0; t < 4 * QN; t++) {
                        float term = ldexpf((float)p[t], (int)w[t] + (int)sbb - 254 - 12);
                        if (w[t] == SCALE_NAN || sbb == SCALE_NAN) term = __uint_as_float(0x7FC00000u);
                        acc[x][t] += term;
                    }
                }
            }
        }
        wave_lds_sync8();   // tiles and lines are read before the next chunk is parked in them
    }

    // ---- the eight partial sums, always w0 + w1 + ... + w7; the staging tiles are done with
    __syncthreads();
    float *red = reinterpret_cast<float *>(lds);
    if (wave > 0) {
#pragma unroll
        for (int x = 0; x < MT; x++)
#pragma unroll
            for (int t = 0; t < 4 * QN; t++) red[(((wave - 1) * MT + x) * 16 + t) * 64 + lane] = acc[x][t];
    }
    __syncthreads();
    if (wave != 0) return;
    const int64_t col = n0 + i;
#pragma unroll
    for (int x = 0; x < MT; x++)
#pragma unroll
        for (int t = 0; t < 4 * QN; t++) {
            float v = acc[x][t];
#pragma unroll
            for (int w = 0; w < I8_WAVES - 1; w++) v += red[((w * MT + x) * 16 + t) * 64 + lane];
            const int64_t r = m0 + 32 * x + 8 * (t / 4) + 4 * g + (t % 4);
            if (r < M && col < N) {
                if (CDT == DT_F32) reinterpret_cast<float *>(C)[r * ldc + col] = v;
                else reinterpret_cast<uint16_t *>(C)[r * ldc + col] = (uint16_t)f32_to_bf16_bits(v);
            }
        }
}

template <int MT, int QN>
static hipError_t launch_int8_lds(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, const uint8_t *Be,
                                  const uint8_t *Bs, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    const dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 32 * MT - 1) / (32 * MT)));
    if (c_dt == DT_F32)
        hipLaunchKernelGGL((gemm_int8_lds_kernel<MT, QN, DT_F32>), grid, dim3(64 * I8_WAVES), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
    else
        hipLaunchKernelGGL((gemm_int8_lds_kernel<MT, QN, DT_BF16>), grid, dim3(64 * I8_WAVES), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
    return hipGetLastError();
}

static hipError_t launch_int8_direct(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, const uint8_t *Be,
                                     const uint8_t *Bs, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    const dim3 grid((unsigned)((N + 63) / 64), (unsigned)((M + 63) / 64));
    if (c_dt == DT_F32) hipLaunchKernelGGL((gemm_int8_kernel<DT_F32>), grid, dim3(256), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
    else hipLaunchKernelGGL((gemm_int8_kernel<DT_BF16>), grid, dim3(256), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
    return hipGetLastError();
}

static hipError_t launch_int8_repair(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, const uint8_t *Be,
                                     const uint8_t *Bs, void *C, int c_dt, int64_t ldc, const uint32_t *range, unsigned n_a, unsigned n_b,
                                     hipStream_t st)
{
    const int64_t tiles = ((N + 63) / 64) * ((M + 63) / 64);
    const dim3 grid((unsigned)(tiles < 512 ? tiles : 512));
    unsigned limit = 379;                                      // see int8_widen_kernel
    for (int64_t k = 1; k < K; k *= 2) limit--;
    if (c_dt == DT_F32)
        hipLaunchKernelGGL((gemm_int8_repair_kernel<DT_F32>), grid, dim3(256), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc, range, n_a, n_b, limit);
    else
        hipLaunchKernelGGL((gemm_int8_repair_kernel<DT_BF16>), grid, dim3(256), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc, range, n_a, n_b, limit);
    return hipGetLastError();
}

// Scratch memory of launch_int8_widened: a word per work-group of int8_widen_kernel, then the values of A and of B
struct Widened {
    unsigned groups_a, groups_b;
    size_t a_at, b_at, bytes;
    Widened(int64_t M, int64_t N, int64_t K)
    {
        auto up256 = [](size_t n) { return (n + 255) & ~(size_t)255; };
        groups_a = (unsigned)((M * K + WIDEN_ELEMS - 1) / WIDEN_ELEMS);
        groups_b = (unsigned)((N * K + WIDEN_ELEMS - 1) / WIDEN_ELEMS);
        a_at = up256(((size_t)groups_a + groups_b) * 4);
        b_at = a_at + up256((size_t)M * (size_t)K * 2);
        bytes = up256(b_at + (size_t)N * (size_t)K * 2);
    }
};

// Whole 256 x 256 tiles that fill much of the chip: scratch memory has always been part of their product
static bool int8_whole_tiles(int64_t M, int64_t N, int64_t K)
{
    const int64_t tiles = (M / 256) * (N / 256);
    return M % 256 == 0 && N % 256 == 0 && K >= 128 && (tiles >= 96 || (tiles >= 64 && K < 1024));
}

// Whether the bf16 values are worth their making for other sizes, which have kernels without scratch memory.  Widening takes 3 bytes an
// element at 4 TB/s and two more launches; and where the library allocates by itself, the memory goes back to the driver whenever
// the device is waited for, so that a call that is waited for takes 30 to 40 us more, and up to 250 from 64 MB on.  The lines lie where a call
// is not slower even so, one allocation in many apart.  us, the kernels without scratch / with the caller's scratch / allocated by the library and waited for
// (in brackets the first of them waited for):
//  - the staged kernel runs its 64 x 32 tiles in rounds of 256, 5.4 + 2.85 K / 1024 us each: 748 x 2432 x 1408 43 / 25 / 65 (55), 353 x 4618 x 4608
//    78 / 53 / 96 (89), 669 x 7461 x 1024 90 / 53 / 89 (100), 936 x 8448 x 2176 205 / 77 / 125 (218); beyond 64 MB 6690 x 801 x 7168 293 / 156 / 334
//    (298), 1719 x 9664 x 7168 792 / 373 / 466 (804).  Up to 128 rows it reads the weights once, the values are read twice and written.
//  - the direct kernel (short or odd K) takes some 24 us for 2^31 products: 4806 x 1099 x 896 66 / 46 / 84 (77), 2847 x 2112 x 1248 87 / 47 /
//    91 (98), 2908 x 4992 x 896 133 / 62 / 106 (142).  Short K is C's write, in rows whose ends are no whole 16 bytes above all:
//    3121 x 6304 x 512 121 / 55 / 96 (131), 1744 x 9463 x 512 103 / 89 / 131 (113); 5680 x 9728 x 320 155 / 92 / 128 (167), 7333 x 1948 x 256 46 / 64 / 105
//    (58), 5251 x 4911 x 96 30 / 101 / 116 (43).
static bool int8_widened_pays(int64_t M, int64_t N, int64_t K)
{
    if (M <= 128) return false;
    const bool staged = K % 128 == 0 && K >= 1024;
    const int64_t without = staged ? (((M + 63) / 64) * ((N + 31) / 32) + 255) / 256 * (5400 + K * 2783 / 1000) / 1000      // us
                                   : M * N * K / (((int64_t)1 << 31) / 24);
    const int64_t least = Widened(M, N, K).bytes >= (size_t)64 << 20 ? 450 : K >= 1024 || (K >= 512 && N % 8 == 0) ? 100 : 190;
    return K >= 256 && without >= least;
}

static bool int8_widened(int64_t M, int64_t N, int64_t K)
{
    return gemm_bf16_applies(M, N, K) && (int8_whole_tiles(M, N, K) || int8_widened_pays(M, N, K));
}

size_t gemm_int8_workspace(int64_t M, int64_t N, int64_t K) { return int8_widened(M, N, K) ? Widened(M, N, K).bytes : 0; }

// C from the bf16 values of the blocks, in scratch memory (ws: Widened::bytes)
static hipError_t launch_int8_widened(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, const uint8_t *Be,
                                      const uint8_t *Bs, void *C, int c_dt, int64_t ldc, uint8_t *ws, hipStream_t st)
{
    const Widened at(M, N, K);
    uint32_t *range = reinterpret_cast<uint32_t *>(ws);
    uint16_t *Aw = reinterpret_cast<uint16_t *>(ws + at.a_at), *Bw = reinterpret_cast<uint16_t *>(ws + at.b_at);
    hipLaunchKernelGGL(int8_widen_kernel, dim3(at.groups_a + at.groups_b), dim3(256), 0, st, Ae, As, M * K, Be, Bs, N * K, Aw, Bw, range, at.groups_a);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_gemm_bf16(M, N, K, Aw, Bw, C, c_dt, ldc, !int8_whole_tiles(M, N, K), st);
    if (e == hipSuccess) e = launch_int8_repair(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, range, at.groups_a, at.groups_b, st);
    return e;
}

hipError_t launch_gemm_int8(int64_t M, int64_t N, int64_t K, const uint8_t *Ae, const uint8_t *As, const uint8_t *Be,
                            const uint8_t *Bs, void *C, int c_dt, int64_t ldc, hipStream_t st)
{
    // Routes, picked by measurement (bf16 output; TOP/s = 2 M N K / time):
    //  - the product of the bf16 values (int8_widened_pays): 8192 x 4096 x 4096 1100 to 1210 TOP/s, 4096^3 960 to 1110, 1000 x 4096 x 4096 530 to 560;
    //  - the LDS-staged shared-K kernel (K a multiple of 128): about 250 TOP/s when K is long, falling with K (each tile's eight
    //    partial sums cost the same whatever K is): 256 x 4096 x 4096 34 us, 1000 x 1000 x 1024 18;
    //  - the unstaged shared-K kernel for few rows or few tiles when K is not a multiple of 128;
    //  - the direct kernel for everything else (short K, odd shapes): 80-170 TOP/s.
    // By shape alone, with or without a caller's workspace: the same product gives the same bits through every entry point.  Only
    // where the memory pool has none, sizes other than whole tiles, which need no scratch elsewhere, take the kernel without (other
    // sums of the same blocks).
    if (int8_widened(M, N, K)) {
        uint8_t *ws = nullptr;
        hipError_t e = ws_acquire(Widened(M, N, K).bytes, st, &ws);
        if (e == hipSuccess) {
            e = launch_int8_widened(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, ws, st);
            const hipError_t f = ws_release(ws, st);
            return e != hipSuccess ? e : f;
        }
        if (e != hipErrorOutOfMemory || int8_whole_tiles(M, N, K)) return e;
    }
    if (M > 0 && N > 0 && K % 128 == 0 && (M <= 128 ? K >= 8 * BLOCK : K >= 1024) && (M + 63) / 64 <= 65535)
        return M <= 8    ? launch_int8_lds<1, 1>(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, st)
               : M <= 16 ? launch_int8_lds<1, 2>(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, st)
               : M <= 32 ? launch_int8_lds<1, 4>(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, st)
                         : launch_int8_lds<2, 4>(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, st);
    // K not in whole 128-byte pieces: few rows, or so few tiles that the direct kernel would put at most one
    // wave on a SIMD while K is long (256 x 4096 x 4096 81 -> 66 us; with 2048 tiles of 32 x 32 the direct
    // kernel is ahead again, 114 vs 124 us)
    const int64_t tiles32 = ((M + 31) / 32) * ((N + 31) / 32);
    if (M > 0 && N > 0 && ((M <= 128 && K >= 8 * BLOCK) || (tiles32 <= 1024 && K >= 4096))) {
        const dim3 grid((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32));
        if (c_dt == DT_F32)
            hipLaunchKernelGGL((gemm_int8_shared_k_kernel<DT_F32>), grid, dim3(64 * I8_WAVES), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
        else
            hipLaunchKernelGGL((gemm_int8_shared_k_kernel<DT_BF16>), grid, dim3(64 * I8_WAVES), 0, st, M, N, K, Ae, As, Be, Bs, C, ldc);
        return hipGetLastError();
    }
    return launch_int8_direct(M, N, K, Ae, As, Be, Bs, C, c_dt, ldc, st);
}

}  // namespace mx
