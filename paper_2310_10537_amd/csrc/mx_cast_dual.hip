// Dual-axis MX cast (Algorithm 1, Section 3 of arXiv 2310.10537, applied along both
// axes of one tensor): training needs every tensor cast with its blocks along the
// reduction axis of each GEMM that uses it -- X and X^T, W and W^T, dY and dY^T
// (Section 4.1: the two casts differ) -- so one pass over the source emits
// both MX tensors.  Source bytes are read once instead of twice.
//
// A work-group stages a 128-row x 64-column tile in LDS with coalesced 16-byte
// row loads.  Chunk c (16 bytes) of row r sits at chunk position
// (c + r + 2 * (r / 32)) % 8 of its 128-byte LDS row, which keeps all three
// access patterns free of bank conflicts: the staging stores (8 lanes cover a
// row), the row reads (a lane takes four consecutive chunks of its row; eight
// lanes = four rows x two halves hit eight different positions) and the column
// reads (sixteen adjacent columns of one row for each of four row blocks, the
// row blocks 32 bytes apart).
//   row part    thread t: row t / 2, columns 32 * (t % 2) .. + 31      -> axis-1 output
//   column part thread t: column t / 4, rows 32 * (t % 4) .. + 31      -> axis-0 output
// Both use the block cast of the stand-alone kernels, so each output is
// bit-identical to what mx_quantize writes for that axis.
#include "mx_convert.hpp"
#include "mx_launch.hpp"

namespace mx {

constexpr int DUAL_R = 128, DUAL_C = 64;
constexpr int DUAL_SG_F32 = 16;     // column strips that the Float32 kernel walks abreast

template <int w>
__device__ __forceinline__ void store_block(uint8_t *o, const uint32_t *out)
{
    if constexpr (w == 8) {
        st16(o, make_uint4(out[0], out[1], out[2], out[3]));
        st16(o + 16, make_uint4(out[4], out[5], out[6], out[7]));
    } else if constexpr (w == 6) {
        *reinterpret_cast<uint2 *>(o) = make_uint2(out[0], out[1]);
        *reinterpret_cast<uint2 *>(o + 8) = make_uint2(out[2], out[3]);
        *reinterpret_cast<uint2 *>(o + 16) = make_uint2(out[4], out[5]);
    } else {
        st16(o, make_uint4(out[0], out[1], out[2], out[3]));
    }
}

// Tile tile_id of the walk: groups of sg adjacent column strips (the last one narrower), strips fastest.
template <int TC>
__device__ __forceinline__ void dual_tile(int64_t tile_id, int64_t row_tiles, int64_t n_tiles, int64_t sg, int64_t &c0, int64_t &r0)
{
    const uint32_t id = (uint32_t)tile_id, rt = (uint32_t)row_tiles, g = (uint32_t)sg;      // n_tiles < 2^31 (launcher)
    const uint32_t strips = (uint32_t)n_tiles / rt, grp = id / (g * rt), in = id - grp * (g * rt);
    const uint32_t width = min(g, strips - grp * g), row = in / width;
    c0 = (int64_t)(grp * g + in - row * width) * TC;
    r0 = (int64_t)row * DUAL_R;
}

// WHOLE: rows a multiple of 128, cols a multiple of TC = 64 or 128 (no bounds checks).  Otherwise rows and cols are
// multiples of 32 (the entry point's rule), TC = 64, and the tiles at the edges are partial.  With 128-column tiles a
// row holds 16 chunks and the same rotation works modulo 16; the row part then writes whole lines (four
// blocks per row, two per thread), the column part two columns per thread.
template <int FMT, int RND, int TC, bool WHOLE>
__global__ __launch_bounds__(256) void cast_dual_bf16_kernel(const uint16_t *__restrict__ src, int64_t rows, int64_t cols,
                                                             int64_t ld, uint8_t *__restrict__ e1, uint8_t *__restrict__ s1,
                                                             uint8_t *__restrict__ e0, uint8_t *__restrict__ s0,
                                                             int64_t row_tiles, int64_t n_tiles, int64_t per_xcd, int64_t sg)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    constexpr int PITCH = TC * 2, NCH = TC / 8;          // bytes and 16-byte chunks per tile row
    __shared__ __attribute__((aligned(16))) uint8_t tile[DUAL_R * PITCH];
    __shared__ __attribute__((aligned(16))) uint32_t xch[w == 6 ? 256 * 6 : 4];   // FP6 column codes on their way out
    const int t = threadIdx.x;
    // XCD-first tile order: each XCD owns a contiguous run of tiles
    const int64_t tile_id = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || tile_id >= n_tiles) return;   // uniform over the work-group
    // Groups of sg adjacent column strips are walked strips-fastest: the row-part pieces a 64-column
    // tile writes (64 / 48 / 32 bytes per row) are then completed to whole lines by the
    // neighbouring strips while they are still in L2 (measured: 188 -> 146 us on a
    // 16384 x 8192 FP6 cast), and the column-part pieces still follow each other closely.
    int64_t c0, r0;
    dual_tile<TC>(tile_id, row_tiles, n_tiles, sg, c0, r0);

    // ---- coalesced loads: NCH lanes per row segment, all in flight before the first LDS write
    {
        constexpr int RPP = 256 / NCH, NP = DUAL_R / RPP;
        const int lr = t / NCH, lc = t % NCH;
        uint4 v[NP];
#pragma unroll
        for (int p = 0; p < NP; p++) {
            if (WHOLE || (r0 + p * RPP + lr < rows && c0 + lc * 8 < cols)) v[p] = ld16_nt(src + (r0 + p * RPP + lr) * ld + c0 + lc * 8);
            else v[p] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < NP; p++) {
            const int r = p * RPP + lr;
            *reinterpret_cast<uint4 *>(tile + r * PITCH + (((lc + r + 2 * (r >> 5)) & (NCH - 1)) << 4)) = v[p];
        }
    }
    __syncthreads();

    const int64_t n_cb = cols / BLOCK, n_rb = rows / BLOCK;
    // ---- row part: thread t takes row t / 2 and half t % 2 of its columns (one or two blocks)
    {
        constexpr int NBR = TC / 64;
        const int r = t >> 1, b = t & 1;
        const uint8_t *rowp = tile + r * PITCH;
        const int rot = r + 2 * (r >> 5);
        uint32_t sc = 0;
        uint32_t o6[12];
#pragma unroll
        for (int j = 0; j < NBR; j++) {
            const int bb = b * NBR + j;
            uint32_t d[16];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint4 q = *reinterpret_cast<const uint4 *>(rowp + (((4 * bb + i + rot) & (NCH - 1)) << 4));
                d[4 * i] = q.x; d[4 * i + 1] = q.y; d[4 * i + 2] = q.z; d[4 * i + 3] = q.w;
            }
            uint32_t out[w];
            const uint32_t s = quantize_block_bf16<FMT, RND>(d, out);
            const int64_t blk = (r0 + r) * n_cb + c0 / BLOCK + bb;
            if constexpr (w == 6 && NBR == 2) {
                // a thread's two FP6 blocks are 48 consecutive, 16-byte aligned bytes: three 16-byte stores
#pragma unroll
                for (int i = 0; i < 6; i++) o6[6 * j + i] = out[i];
                if (j == 1) {
                    uint8_t *o = e1 + (blk - 1) * 24;
                    st16(o, make_uint4(o6[0], o6[1], o6[2], o6[3]));
                    st16(o + 16, make_uint4(o6[4], o6[5], o6[6], o6[7]));
                    st16(o + 32, make_uint4(o6[8], o6[9], o6[10], o6[11]));
                }
            } else if (WHOLE || (r0 + r < rows && c0 / BLOCK + bb < n_cb)) {
                store_block<w>(e1 + blk * (BLOCK * w / 8), out);
                if constexpr (!WHOLE) s1[blk] = (uint8_t)s;
            }
            sc |= s << (8 * j);
        }
        // the blocks of a row sit in two adjacent lanes: one 16- or 32-bit store
        const int64_t blk0 = (r0 + r) * n_cb + c0 / BLOCK;
        const uint32_t sall = sc | ((uint32_t)__shfl_down((int)sc, 1) << (8 * NBR));
        if (WHOLE && b == 0) {
            if constexpr (NBR == 1) *reinterpret_cast<uint16_t *>(s1 + blk0) = (uint16_t)sall;
            else *reinterpret_cast<uint32_t *>(s1 + blk0) = sall;
        }
    }
    // ---- column part: thread t takes row block t % 4 of column t / 4 (and of column t / 4 + 64)
#pragma unroll
    for (int q = 0; q < TC / 64; q++) {
        const int c = (t >> 2) + 64 * q, rb = t & 3;
        uint32_t d[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            // rows rb*32 + 2i and + 2i + 1: chunk c / 8 of the row, rotated like the stores
            const int ra = 2 * i, rbw = 2 * i + 1;
            const uint32_t lo = *reinterpret_cast<const uint16_t *>(tile + (rb * 32 + ra) * PITCH + ((((c >> 3) + ra + 2 * rb) & (NCH - 1)) << 4) + (c & 7) * 2);
            const uint32_t hi = *reinterpret_cast<const uint16_t *>(tile + (rb * 32 + rbw) * PITCH + ((((c >> 3) + rbw + 2 * rb) & (NCH - 1)) << 4) + (c & 7) * 2);
            d[i] = lo | (hi << 16);
        }
        uint32_t out[w];
        const uint32_t s = quantize_block_bf16<FMT, RND>(d, out);
        const int64_t blk = (c0 + c) * n_rb + r0 / BLOCK + rb;
        if constexpr (!WHOLE) {
            if (c0 + c < cols && r0 / BLOCK + rb < n_rb) {
                store_block<w>(e0 + blk * (BLOCK * w / 8), out);
                s0[blk] = (uint8_t)s;
            }
            continue;
        }
        if constexpr (w == 6) {
            // the four lanes of a column hold 96 consecutive, 16-byte aligned output bytes; through LDS
            // (a wave-private exchange: lanes of a quad are in one wave) they leave as six 16-byte stores
            uint32_t *x = xch + (t & ~3) * 6;
#pragma unroll
            for (int i = 0; i < 6; i += 2) *reinterpret_cast<uint2 *>(x + rb * 6 + i) = make_uint2(out[i], out[i + 1]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint8_t *oq = e0 + (blk - rb) * 24;
            st16(oq + rb * 16, *reinterpret_cast<const uint4 *>(x + rb * 4));
            if (rb < 2) st16(oq + 64 + rb * 16, *reinterpret_cast<const uint4 *>(x + 16 + rb * 4));
            if (q + 1 < TC / 64) {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        } else {
            store_block<w>(e0 + blk * (BLOCK * w / 8), out);
        }
        const uint32_t s4 = s | ((uint32_t)__shfl_down((int)s, 1) << 8) | ((uint32_t)__shfl_down((int)s, 2) << 16) |
                            ((uint32_t)__shfl_down((int)s, 3) << 24);
        if (rb == 0) *reinterpret_cast<uint32_t *>(s0 + blk) = s4;
    }
}

// ---------------------------------------------------------------------------
// Float32 source (master weights after an optimizer step; rows and cols multiples of 32).  Bound by HBM: 4 bytes in
// and 2 * (bits / 8 + 1 / 32) out per element; two casts read the source twice (4096 x 11008 -> E4M3: 81 us; this kernel 54 us,
// 5.1 TB/s).  Remainders of a tile take the form with bounds checks, of either source type, instead of two casts.
// The plan is that of the bf16 kernel on a 128-row x 64-column tile of 16 chunks a row (256 bytes, one pass over the 64 banks).  Chunk
// q of row r sits at position (q + r + 4 * (r / 32)) % 16: the row reads (16 lanes = eight rows x two halves, 16 bytes each)
// and the column reads (16 columns = four chunks of one row in each of four row blocks) hit 16 different positions.
// ---------------------------------------------------------------------------
constexpr int DUAL_PITCH = 64;                       // dwords

template <int FMT, int RND, bool WHOLE>
__global__ __launch_bounds__(256) void cast_dual_f32_kernel(const float *__restrict__ src, int64_t rows, int64_t cols, int64_t ld,
                                                            uint8_t *__restrict__ e1, uint8_t *__restrict__ s1, uint8_t *__restrict__ e0,
                                                            uint8_t *__restrict__ s0, int64_t row_tiles, int64_t n_tiles, int64_t per_xcd,
                                                            int64_t sg)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    __shared__ __attribute__((aligned(16))) uint32_t tile[DUAL_R * DUAL_PITCH];
    const int t = threadIdx.x;
    const int64_t tile_id = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || tile_id >= n_tiles) return;   // uniform over the work-group
    int64_t c0, r0;
    dual_tile<DUAL_C>(tile_id, row_tiles, n_tiles, sg, c0, r0);
    {
        const int lr = t >> 4, lc = t & 15;
        uint4 v[DUAL_R / 16];
#pragma unroll
        for (int p = 0; p < DUAL_R / 16; p++) {
            if (WHOLE || (r0 + p * 16 + lr < rows && c0 + lc * 4 < cols)) v[p] = ld16_nt(src + (r0 + p * 16 + lr) * ld + c0 + lc * 4);
            else v[p] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < DUAL_R / 16; p++) {
            const int r = p * 16 + lr;
            *reinterpret_cast<uint4 *>(tile + r * DUAL_PITCH + (((lc + r + 4 * (r >> 5)) & 15) << 2)) = v[p];
        }
    }
    __syncthreads();

    const int64_t n_cb = cols / BLOCK, n_rb = rows / BLOCK;
    // ---- row part: thread t takes row t / 2, columns 32 * (t % 2) .. + 31
    {
        const int r = t >> 1, b = t & 1, rot = 8 * b + r + 4 * (r >> 5);
        const uint32_t *rowp = tile + r * DUAL_PITCH;
        uint32_t v[32], out[w];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const uint4 q = *reinterpret_cast<const uint4 *>(rowp + (((i + rot) & 15) << 2));
            v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
        }
        const uint32_t s = quantize_block_f32<FMT, RND>(v, [&](int i) { return rowp[((((i >> 2) + rot) & 15) << 2) + (i & 3)]; }, out);
        const int64_t blk = (r0 + r) * n_cb + c0 / BLOCK + b;
        if (WHOLE || (r0 + r < rows && c0 / BLOCK + b < n_cb)) store_block<w>(e1 + blk * (BLOCK * w / 8), out);
        if constexpr (WHOLE) {                       // the two blocks of a row sit in adjacent lanes, an even number of blocks in a row
            const uint32_t s2 = s | ((uint32_t)__shfl_down((int)s, 1) << 8);
            if (b == 0) *reinterpret_cast<uint16_t *>(s1 + blk) = (uint16_t)s2;
        } else if (r0 + r < rows && c0 / BLOCK + b < n_cb) {
            s1[blk] = (uint8_t)s;
        }
    }
    // ---- column part: thread t takes column t / 4, rows 32 * (t % 4) .. + 31
    {
        const int c = t >> 2, rb = t & 3, rot = (c >> 2) + 4 * rb;
        const uint32_t *colp = tile + rb * 32 * DUAL_PITCH + (c & 3);
        auto at = [&](int i) { return colp[i * DUAL_PITCH + (((i + rot) & 15) << 2)]; };
        uint32_t v[32], out[w];
#pragma unroll
        for (int i = 0; i < 32; i++) v[i] = at(i);
        const uint32_t s = quantize_block_f32<FMT, RND>(v, at, out);
        const int64_t blk = (c0 + c) * n_rb + r0 / BLOCK + rb;
        if (WHOLE || (c0 + c < cols && r0 / BLOCK + rb < n_rb)) store_block<w>(e0 + blk * (BLOCK * w / 8), out);
        if constexpr (WHOLE) {
            const uint32_t s4 = s | ((uint32_t)__shfl_down((int)s, 1) << 8) | ((uint32_t)__shfl_down((int)s, 2) << 16) |
                                ((uint32_t)__shfl_down((int)s, 3) << 24);
            if (rb == 0) *reinterpret_cast<uint32_t *>(s0 + blk) = s4;
        } else if (c0 + c < cols && r0 / BLOCK + rb < n_rb) {
            s0[blk] = (uint8_t)s;
        }
    }
}

// Launches kernel(grid, tiles...) over tiles of 128 rows x tc columns; strips are walked sg abreast.
template <typename F>
static hipError_t dual_grid(int64_t rows, int64_t cols, int tc, F go)
{
    const int64_t row_tiles = (rows + DUAL_R - 1) / DUAL_R, n_tiles = row_tiles * ((cols + tc - 1) / tc), per_xcd = (n_tiles + 7) / 8;
    if (per_xcd * 8 > 0x7FFFFFFF || row_tiles > 0x7FFFFFF) return hipErrorNotSupported;       // dual_tile counts in 32 bits
    go(dim3((unsigned)(per_xcd * 8)), row_tiles, n_tiles, per_xcd);
    return hipGetLastError();
}

template <int FMT, int RND>
static hipError_t launch_dual_r(const void *src, int src_dt, int64_t rows, int64_t cols, int64_t ld, uint8_t *e1, uint8_t *s1,
                                uint8_t *e0, uint8_t *s0, hipStream_t st)
{
    const bool whole = rows % DUAL_R == 0 && cols % DUAL_C == 0;
    // bf16: 128-column tiles once they still give every compute unit several work-groups
    const int tc = src_dt == DT_BF16 && whole && cols % 128 == 0 && (rows / DUAL_R) * (cols / 128) >= 1024 ? 128 : DUAL_C;
    return dual_grid(rows, cols, tc, [&](dim3 grid, int64_t row_tiles, int64_t n_tiles, int64_t per_xcd) {
#define MX_DUAL(KERNEL, T, SG) hipLaunchKernelGGL(KERNEL, grid, dim3(256), 0, st, static_cast<const T *>(src), rows, cols, ld, e1, s1, e0, s0, row_tiles, n_tiles, per_xcd, (int64_t)(SG))
        if (src_dt == DT_F32) {
            if (whole) MX_DUAL((cast_dual_f32_kernel<FMT, RND, true>), float, DUAL_SG_F32);
            else MX_DUAL((cast_dual_f32_kernel<FMT, RND, false>), float, DUAL_SG_F32);
        } else if (tc == 128) {
            MX_DUAL((cast_dual_bf16_kernel<FMT, RND, 128, true>), uint16_t, 8);
        } else if (whole) {
            MX_DUAL((cast_dual_bf16_kernel<FMT, RND, DUAL_C, true>), uint16_t, 16);
        } else {
            MX_DUAL((cast_dual_bf16_kernel<FMT, RND, DUAL_C, false>), uint16_t, 16);
        }
#undef MX_DUAL
    });
}

template <int FMT>
static hipError_t launch_dual_fmt(int rnd, const void *src, int src_dt, int64_t rows, int64_t cols, int64_t ld, uint8_t *e1, uint8_t *s1,
                                  uint8_t *e0, uint8_t *s0, hipStream_t st)
{
    return rnd == ROUND_RNE ? launch_dual_r<FMT, ROUND_RNE>(src, src_dt, rows, cols, ld, e1, s1, e0, s0, st)
                            : launch_dual_r<FMT, ROUND_HALF_AWAY>(src, src_dt, rows, cols, ld, e1, s1, e0, s0, st);
}

// One pass for both axes; two ordinary casts (same bytes) for the rounding modes without hardware converts, and for 32 long rows of
// Float32 to 8 bits, which fill a quarter of a tile (32 x 582272 E5M2: one pass 43 us, two casts 38).
hipError_t launch_cast_dual(const void *src, int src_dt, int64_t rows, int64_t cols, int64_t ld, int fmt, int rnd,
                            uint8_t *e1, uint8_t *s1, uint8_t *e0, uint8_t *s0, hipStream_t st)
{
    const bool quarter = src_dt == DT_F32 && fmt_bits(fmt) == 8 && rows == BLOCK && cols >= ((int64_t)1 << 17);
    if (!quarter && (rnd == ROUND_RNE || rnd == ROUND_HALF_AWAY)) {
        hipError_t e;
        switch (fmt) {
            case FP8_E4M3: e = launch_dual_fmt<FP8_E4M3>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
            case FP8_E5M2: e = launch_dual_fmt<FP8_E5M2>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
            case FP6_E3M2: e = launch_dual_fmt<FP6_E3M2>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
            case FP6_E2M3: e = launch_dual_fmt<FP6_E2M3>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
            case FP4_E2M1: e = launch_dual_fmt<FP4_E2M1>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
            default:       e = launch_dual_fmt<INT8>(rnd, src, src_dt, rows, cols, ld, e1, s1, e0, s0, st); break;
        }
        if (e != hipErrorNotSupported) return e;
    }
    hipError_t e = launch_cast(src, src_dt, rows, cols, ld, 1, fmt, rnd, e1, s1, st);
    if (e != hipSuccess) return e;
    return launch_cast(src, src_dt, rows, cols, ld, 0, fmt, rnd, e0, s0, st);
}

}  // namespace mx
