// Bandwidth-oriented MX cast kernels for bf16 sources (Algorithm 1, Section 3 of
// arXiv 2310.10537) on gfx950.  Both are pure streaming kernels bound by HBM:
// per element they read 2 bytes and write bits/8 + 1/32 bytes.
//
//   cast_row_bf16_kernel   blocks along the contiguous axis.  A wave takes 2048
//       consecutive elements as four fully coalesced 16-byte-per-lane loads
//       (1 KB per instruction).  8-bit and 4-bit formats convert in place: four
//       adjacent lanes share a block, the block maximum is a packed-u16 max
//       finished with two DPP quad permutes.  FP6 converts 32 elements per
//       instruction, so the wave transposes its 64 blocks through a private LDS
//       region until each lane owns one block.  Scale bytes (and FP6 codes) are
//       staged in LDS so that they leave as 16-byte stores.
//   cast_col_bf16_kernel   blocks along dimension 0, output written as the cast of
//       the transpose.  A work-group stages a [128 rows x 128 (or 64) columns] tile in LDS
//       with coalesced row loads (rows rotated by 32 bytes per 32-row block so
//       that column reads are bank-conflict free); each lane then reads one
//       column of one 32-row block -- the block maximum is in-lane -- and the four
//       lanes of a column write one contiguous 128 / 96 / 64-byte output line.
#include "mx_convert.hpp"
#include "mx_launch.hpp"

namespace mx {

// Lanes of one wave exchange data through LDS without a work-group barrier: LDS
// operations of a wave execute in order, so it is enough to keep the compiler
// from moving accesses across this point and to wait for the wave's own writes.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Row cast
// ---------------------------------------------------------------------------
constexpr int ROW_CHUNKS = 4;                 // 16-byte loads in flight per lane (8 measured the same, 16 slower)
constexpr int ROW_WAVE_ELEMS = 64 * 8 * ROW_CHUNKS;   // 2048 elements = 64 blocks per wave

// FLAT: dense rows of whole blocks, one run of n_elems elements.  Otherwise the rows are those of `geom`
// (padded pitch, a batch of matrices, a partial last block that is filled up with zeros) and n_elems counts
// the fill: the outputs are one run in either form.  (5120 x 5000 -> E4M3: 14 us, 5.4 TB/s; the generic
// kernel, which rows of partial blocks used to take, 28 us.)  WHOLE: every wave's elements lie inside the tensor.
template <int FMT, int RND, bool FLAT, bool WHOLE = false, int CH = ROW_CHUNKS>
__global__ __launch_bounds__(256) void cast_row_bf16_kernel(const uint16_t *__restrict__ src, RowGeom geom,
                                                            uint8_t *__restrict__ elems, uint8_t *__restrict__ scales,
                                                            int64_t n_elems)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    constexpr bool SIX = (w == 6);
    // per wave: FP6 needs 64 blocks x 80 bytes (padded) for the transpose; everyone needs 64 scale bytes
    static_assert(!SIX || CH == 4, "the FP6 transpose gives lane L block L of 64");
    constexpr int LDS_PER_WAVE = SIX ? 64 * 80 : 16 * CH;
    constexpr int WAVE_ELEMS = 512 * CH;
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[4 * LDS_PER_WAVE];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint8_t *lds = lds_all + wave * LDS_PER_WAVE;

    const int64_t wave_id = (int64_t)blockIdx.x * 4 + wave;
    const int64_t e0 = wave_id * WAVE_ELEMS;          // first element of this wave
    if (!WHOLE && e0 >= n_elems) return;                  // whole wave out of range
    const int64_t blk0 = e0 / BLOCK;                      // first block of this wave

    // ---- coalesced loads: chunk u, lane l -> elements e0 + u*512 + l*8 .. +7
    uint32_t d[CH][4];
    bool valid[CH];
#pragma unroll
    for (int u = 0; u < CH; u++) {
        const int64_t e = e0 + u * 512 + lane * 8;
        valid[u] = WHOLE || e < n_elems;
        uint4 t = make_uint4(0, 0, 0, 0);
        if constexpr (FLAT) {
            if (valid[u]) t = ld16_nt(src + e);
        } else if (valid[u]) {
            int n;
            const uint16_t *g = src + geom.at((uint32_t)(e >> 3), 8, n);
            if (n == 8) {
                t = ld16_nt(g);
            } else if (n > 0) {
                uint32_t h[8];
#pragma unroll
                for (int i = 0; i < 8; i++) h[i] = i < n ? g[i] : 0u;
                t = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
            }
        }
        d[u][0] = t.x; d[u][1] = t.y; d[u][2] = t.z; d[u][3] = t.w;
    }

    if constexpr (!SIX) {
        constexpr int OD = 8 * w / 32;   // output dwords per lane per chunk (2 or 1)
#pragma unroll
        for (int u = 0; u < CH; u++) {
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) m = pk_absmax(m, d[u][i]);
            uint32_t amax16 = group_max<4>(pk_hmax(m));
            uint32_t s = scale_from_bf16_max<FMT>(amax16);
            uint32_t out[OD];
            if (fast_ok(amax16, s)) {
                convert_bf16_fast<FMT, RND, 4>(d[u], s, out);
            } else {
                // exact path; the condition is uniform over the four lanes of the block
                uint32_t v[8];
                widen_bf16<4>(d[u], v);
                uint32_t amax = 0;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    uint32_t k = amax_key<FMT>(v[i]);
                    amax = amax > k ? amax : k;
                }
                amax = group_max<4>(amax);
                s = scale_byte<FMT>(amax);
                encode_exact<FMT, RND, 8>(v, s, out);
            }
            if (valid[u]) {
                uint8_t *o = elems + (e0 + u * 512 + lane * 8) * w / 8;
                if constexpr (OD == 2) *reinterpret_cast<uint2 *>(o) = make_uint2(out[0], out[1]);
                else *reinterpret_cast<uint32_t *>(o) = out[0];
            }
            if ((lane & 3) == 0) lds[u * 16 + (lane >> 2)] = (uint8_t)s;   // block u*16 + lane/4 of this wave
        }
    } else {
        // ---- FP6: transpose so that lane L owns block L of the wave (chunk L/16, quad L%16)
#pragma unroll
        for (int u = 0; u < CH; u++) {
            const int b = u * 16 + (lane >> 2);
            *reinterpret_cast<uint4 *>(lds + b * 80 + (lane & 3) * 16) = make_uint4(d[u][0], d[u][1], d[u][2], d[u][3]);
        }
        wave_lds_sync();
        uint32_t blk[16];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            uint4 t = *reinterpret_cast<const uint4 *>(lds + lane * 80 + j * 16);
            blk[4 * j] = t.x; blk[4 * j + 1] = t.y; blk[4 * j + 2] = t.z; blk[4 * j + 3] = t.w;
        }
        uint32_t out[6];
        const uint32_t s = quantize_block_bf16<FMT, RND>(blk, out);
        wave_lds_sync();
        // codes back through LDS: 64 blocks x 24 bytes = 1536 contiguous bytes, then the scale bytes
        uint32_t *l32 = reinterpret_cast<uint32_t *>(lds);
#pragma unroll
        for (int i = 0; i < 6; i++) l32[lane * 6 + i] = out[i];
        lds[1536 + lane] = (uint8_t)s;
        wave_lds_sync();
        const int64_t n_blk_valid = WHOLE ? 64 : (n_elems - e0) / BLOCK;   // blocks of this wave inside the tensor (>= 1)
        uint8_t *o = elems + blk0 * 24;
        const uint4 a = *reinterpret_cast<const uint4 *>(lds + lane * 16);
        const uint2 c = *reinterpret_cast<const uint2 *>(lds + 1024 + lane * 8);
        if (n_blk_valid >= 64) {
            st16(o + lane * 16, a);
            *reinterpret_cast<uint2 *>(o + 1024 + lane * 8) = c;
        } else {
            const int64_t nbytes = n_blk_valid * 24;           // a multiple of 8
            if (lane * 16 + 16 <= nbytes) st16(o + lane * 16, a);
            else if (lane * 16 + 8 <= nbytes) *reinterpret_cast<uint2 *>(o + lane * 16) = make_uint2(a.x, a.y);
            if (1024 + lane * 8 + 8 <= nbytes) *reinterpret_cast<uint2 *>(o + 1024 + lane * 8) = c;
        }
    }

    // ---- scale bytes: 64 per wave, stored 16 at a time
    wave_lds_sync();
    {
        const uint8_t *sl = SIX ? lds + 1536 : lds;
        const int64_t n_blk_valid = WHOLE ? 16 * CH : (n_elems - e0) / BLOCK;
        if (lane < CH) {
            if ((lane + 1) * 16 <= n_blk_valid) {
                st16(scales + blk0 + lane * 16, *reinterpret_cast<const uint4 *>(sl + lane * 16));
            } else {
                for (int i = lane * 16; i < n_blk_valid && i < lane * 16 + 16; i++) scales[blk0 + i] = sl[i];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Column cast
// ---------------------------------------------------------------------------
constexpr int COL_TILE_R = 128;   // rows of a tile (256 measured slower)
constexpr int COL_TILE_C = 64;    // columns of a tile of the Float32 kernel

// A tile is 128 rows x TC columns, TC = 128 (256-byte row segments, two lines) or 64 for narrow
// tensors.  Work-groups are dealt round-robin to the 8 XCDs, each with its own L2.  Tile
// t = xcd * per_xcd + i, each XCD owning a contiguous run of column strips which it walks down
// the rows: what its work-groups write (128 bytes of codes and 4 scale bytes per column each) is
// consecutive in memory and merges into full lines in that XCD's L2.
// (Measured on the bare access pattern -- loads, LDS tile, stores, no arithmetic -- of an
// 8192 x 8192 tensor: 128 x 64 tiles 38.6 us, 256 x 64 37.2, 128 x 128 35.9, 256 x 128 40.5,
// 64 x 256 37.8; walking several adjacent strips abreast, which paid before the loads became
// non-temporal, now costs 1-2 us.  The kernel runs within 5 % of its pattern.)
// Row and column remainders take the form with bounds checks (5000 x 5120 -> E4M3 22 us, 3.5 TB/s; the
// generic one-lane-per-block kernel, which partial blocks used to take, 43 us), and a batch of matrices
// is one launch (128 matrices of 2048 x 128: a launch each cost 3.5 us apiece).
template <int FMT, int RND, int TC, bool WHOLE>   // WHOLE: every tile lies inside the tensor (no bounds checks)
__global__ __launch_bounds__(256) void cast_col_bf16_kernel(const uint16_t *__restrict__ src, int64_t rows, int64_t cols,
                                                            int64_t ld, uint8_t *__restrict__ elems,
                                                            uint8_t *__restrict__ scales, int64_t row_tiles,
                                                            int64_t n_tiles, int64_t per_xcd, Batch batch)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    constexpr int PITCH = TC * 2;                        // bytes per tile row in LDS
    src += blockIdx.z * batch.src;                       // one launch for all matrices of a batch
    elems += blockIdx.z * batch.elems;
    scales += blockIdx.z * batch.scales;
    __shared__ __attribute__((aligned(16))) uint8_t tile[COL_TILE_R * PITCH];
    __shared__ __attribute__((aligned(16))) uint32_t xch[(w == 6 && WHOLE) ? 256 * 6 : 4];   // FP6 codes on their way out
    const int t = threadIdx.x;
    const int64_t tile_id = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || tile_id >= n_tiles) return;   // uniform over the work-group
    const int64_t ct = tile_id / row_tiles, rt = tile_id % row_tiles;
    const int64_t c0 = ct * TC;
    const int64_t r0 = rt * COL_TILE_R;

    // ---- coalesced loads: TC / 8 lanes per row segment, all in flight before the first LDS write
    constexpr int LPR = TC / 8, RPP = 256 / LPR, NP = COL_TILE_R / RPP;
    const int lr = t / LPR, lc = t % LPR;
    const bool full_cols = WHOLE || c0 + TC <= cols;
    uint4 v[NP];
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int r = p * RPP + lr;                      // row inside the tile
        v[p] = make_uint4(0, 0, 0, 0);
        if (WHOLE || r0 + r < rows) {
            const uint16_t *g = src + (r0 + r) * ld + c0 + lc * 8;
            if (full_cols || c0 + lc * 8 + 8 <= cols) {
                v[p] = ld16_nt(g);
            } else {
                uint16_t h[8];
#pragma unroll
                for (int i = 0; i < 8; i++) h[i] = (c0 + lc * 8 + i < cols) ? g[i] : (uint16_t)0;
                v[p] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
            }
        }
    }
#pragma unroll
    for (int p = 0; p < NP; p++) {
        const int r = p * RPP + lr;
        // rotate the row by 32 bytes per row block: column reads of four adjacent blocks then hit different banks
        *reinterpret_cast<uint4 *>(tile + r * PITCH + ((lc * 16 + (r >> 5) * 32) & (PITCH - 1))) = v[p];
    }
    __syncthreads();

    // ---- lane (column c, row block rb): 32 values down the column, packed in pairs
    // (rows beyond the tensor were staged as zeros: the fill of a partial last block)
    const int64_t n_rb = WHOLE ? rows / BLOCK : (rows + BLOCK - 1) / BLOCK;
    const bool quad = WHOLE || (n_rb & 3) == 0;          // scale dwords are aligned
#pragma unroll
    for (int q = 0; q < TC / 64; q++) {
        const int c = (t >> 2) + 64 * q;
        const int64_t col = c0 + c;
        const int rb = t & 3;
        const int64_t row_blk = r0 / BLOCK + rb;
        const bool valid = WHOLE || (col < cols && row_blk < n_rb);
        const uint8_t *colp = tile + rb * 32 * PITCH + ((c * 2 + rb * 32) & (PITCH - 1));
        uint32_t d[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            uint32_t lo = *reinterpret_cast<const uint16_t *>(colp + (2 * i) * PITCH);
            uint32_t hi = *reinterpret_cast<const uint16_t *>(colp + (2 * i + 1) * PITCH);
            d[i] = lo | (hi << 16);
        }
        uint32_t out[w];
        const uint32_t s = quantize_block_bf16<FMT, RND>(d, out);
        // the four lanes of a column hold four consecutive scale bytes: one dword store when the
        // whole quad is valid and the address is aligned, else byte stores
        const uint32_t s4 = s | ((uint32_t)__shfl_down((int)s, 1) << 8) | ((uint32_t)__shfl_down((int)s, 2) << 16) |
                            ((uint32_t)__shfl_down((int)s, 3) << 24);
        if (valid) {
            uint8_t *o = elems + (col * n_rb + row_blk) * (BLOCK * w / 8);
            if constexpr (w == 8) {
                // (a transpose inside the quad, so that each of the two stores writes 64 consecutive
                // bytes of the column's 128-byte line instead of every second 16, changed nothing
                // measurable: 44.6 against 45.3 us)
                st16(o, make_uint4(out[0], out[1], out[2], out[3]));
                st16(o + 16, make_uint4(out[4], out[5], out[6], out[7]));
            } else if constexpr (w == 6) {
                if constexpr (WHOLE) {
                    // the four lanes of a column hold 96 consecutive output bytes (16-byte aligned: whole
                    // tiles are four blocks deep); through LDS they leave as six 16-byte stores
                    uint32_t *x = xch + (t & ~3) * 6;
#pragma unroll
                    for (int i = 0; i < 6; i += 2) *reinterpret_cast<uint2 *>(x + (t & 3) * 6 + i) = make_uint2(out[i], out[i + 1]);
                    wave_lds_sync();
                    uint8_t *oq = o - (t & 3) * 24;
                    st16(oq + (t & 3) * 16, *reinterpret_cast<const uint4 *>(x + (t & 3) * 4));
                    if ((t & 3) < 2) st16(oq + 64 + (t & 3) * 16, *reinterpret_cast<const uint4 *>(x + 16 + (t & 3) * 4));
                    if (q + 1 < TC / 64) wave_lds_sync();   // the exchange area is written again
                } else {
                    *reinterpret_cast<uint2 *>(o) = make_uint2(out[0], out[1]);
                    *reinterpret_cast<uint2 *>(o + 8) = make_uint2(out[2], out[3]);
                    *reinterpret_cast<uint2 *>(o + 16) = make_uint2(out[4], out[5]);
                }
            } else {
                st16(o, make_uint4(out[0], out[1], out[2], out[3]));
            }
            if (WHOLE || (quad && r0 / BLOCK + 4 <= n_rb)) {   // uniform over the work-group
                if ((t & 3) == 0) *reinterpret_cast<uint32_t *>(scales + col * n_rb + row_blk) = s4;
            } else {
                scales[col * n_rb + row_blk] = (uint8_t)s;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Column cast of a Float32 source (weights are cast from Float32, along the reduction axis of
// their GEMM, i.e. along dimension 0 of a [K][N] tensor).  Same plan
// as the bf16 kernel: coalesced row loads into an LDS tile (here 16 lanes x 16 bytes per 256-byte
// row segment), then lane (column c, row block rb) walks 32 values down its column, and the four
// lanes of a column write its four consecutive blocks.  Row block rb keeps its rows rotated by
// 16 rb columns, so the 64 lanes of a wave (16 columns x 4 row blocks) read 64 different banks.
// The one-lane-per-(block, column) kernel without LDS leaves every output line to eight
// work-groups that run far apart in time: 3.3 TB/s on 8192 x 28672 -> E2M1.
// ---------------------------------------------------------------------------
template <int FMT, int RND, bool WHOLE>   // WHOLE: every tile lies inside the tensor (no bounds checks)
__global__ __launch_bounds__(256) void cast_col_f32_kernel(const float *__restrict__ src, int64_t rows, int64_t cols, int64_t ld,
                                                           uint8_t *__restrict__ elems, uint8_t *__restrict__ scales,
                                                           int64_t row_tiles, int64_t n_tiles, int64_t per_xcd, Batch batch)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    __shared__ __attribute__((aligned(16))) uint32_t tile[COL_TILE_R * COL_TILE_C];   // 32 KB, rows of 64 floats
    src += blockIdx.z * batch.src;
    elems += blockIdx.z * batch.elems;
    scales += blockIdx.z * batch.scales;
    const int t = threadIdx.x;
    const int64_t tile_id = (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int64_t)(blockIdx.x >> 3) >= per_xcd || tile_id >= n_tiles) return;   // uniform over the work-group
    // strips one at a time, as in the bf16 kernel (several abreast cost 3 % with non-temporal loads)
    const int64_t ct = tile_id / row_tiles, rt = tile_id % row_tiles;
    const int64_t c0 = ct * COL_TILE_C, r0 = rt * COL_TILE_R;
    const int lr = t >> 4, lc = t & 15;
    const bool full_cols = WHOLE || c0 + COL_TILE_C <= cols;
    uint4 v[COL_TILE_R / 16];
#pragma unroll
    for (int p = 0; p < COL_TILE_R / 16; p++) {
        v[p] = make_uint4(0, 0, 0, 0);                // rows beyond the tensor: the fill of a partial last block
        if (WHOLE || r0 + p * 16 + lr < rows) {
            const float *g = src + (r0 + p * 16 + lr) * ld + c0 + lc * 4;
            if (full_cols || c0 + lc * 4 + 4 <= cols) {
                v[p] = ld16_nt(g);
            } else {
                uint32_t h[4];
#pragma unroll
                for (int i = 0; i < 4; i++) h[i] = (c0 + lc * 4 + i < cols) ? __float_as_uint(g[i]) : 0u;
                v[p] = make_uint4(h[0], h[1], h[2], h[3]);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < COL_TILE_R / 16; p++) {
        const int r = p * 16 + lr;                    // row inside the tile; its 32-row block is r / 32
        *reinterpret_cast<uint4 *>(tile + r * COL_TILE_C + ((lc * 4 + (r >> 5) * 16) & 63)) = v[p];
    }
    __syncthreads();
    const int c = t >> 2, rb = t & 3;
    const int64_t col = c0 + c, n_rb = WHOLE ? rows / BLOCK : (rows + BLOCK - 1) / BLOCK, row_blk = r0 / BLOCK + rb;
    uint32_t out[w];
    const uint32_t s = quantize_block_lds<FMT, RND>(tile + rb * 32 * COL_TILE_C + ((c + rb * 16) & 63), COL_TILE_C, out);
    const uint32_t s4 = s | ((uint32_t)__shfl_down((int)s, 1) << 8) | ((uint32_t)__shfl_down((int)s, 2) << 16) |
                        ((uint32_t)__shfl_down((int)s, 3) << 24);
    if (!WHOLE && (col >= cols || row_blk >= n_rb)) return;
    uint8_t *o = elems + (col * n_rb + row_blk) * (BLOCK * w / 8);
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
    // four consecutive scale bytes leave as one dword when they exist and the address is aligned
    if (WHOLE || ((n_rb & 3) == 0 && r0 / BLOCK + 4 <= n_rb)) {
        if (rb == 0) *reinterpret_cast<uint32_t *>(scales + col * n_rb + row_blk) = s4;
    } else {
        scales[col * n_rb + row_blk] = (uint8_t)s;
    }
}

// ---------------------------------------------------------------------------
// Launchers.  Return hipErrorNotSupported when the fast path does not apply.
// ---------------------------------------------------------------------------
// gridDim.z walks a batch, at most 65535 matrices per launch
template <typename F>
static hipError_t for_batch(const Batch &b, int src_bytes, const void *src, uint8_t *elems, uint8_t *scales, F go)
{
    for (int64_t i = 0; i < b.n; i += 65535) {
        go((unsigned)(b.n - i < 65535 ? b.n - i : 65535), static_cast<const char *>(src) + i * b.src * src_bytes, elems + i * b.elems,
           scales + i * b.scales);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int FMT, int RND>
static hipError_t launch_col_f32_r(const void *src, int64_t rows, int64_t cols, int64_t ld, uint8_t *elems, uint8_t *scales,
                                   hipStream_t st, const Batch &batch)
{
    const int64_t row_tiles = (rows + COL_TILE_R - 1) / COL_TILE_R, n_tiles = row_tiles * ((cols + COL_TILE_C - 1) / COL_TILE_C);
    const int64_t per_xcd = (n_tiles + 7) / 8;
    if (per_xcd * 8 > 0x7FFFFFFF) return hipErrorNotSupported;
    const bool whole = rows % COL_TILE_R == 0 && cols % COL_TILE_C == 0;
    return for_batch(batch, 4, src, elems, scales, [&](unsigned nz, const char *s, uint8_t *e, uint8_t *sc) {
        const dim3 grid((unsigned)(per_xcd * 8), 1, nz);
        const float *p = reinterpret_cast<const float *>(s);
        if (whole)
            hipLaunchKernelGGL((cast_col_f32_kernel<FMT, RND, true>), grid, dim3(256), 0, st, p, rows, cols, ld, e, sc, row_tiles, n_tiles,
                               per_xcd, batch);
        else
            hipLaunchKernelGGL((cast_col_f32_kernel<FMT, RND, false>), grid, dim3(256), 0, st, p, rows, cols, ld, e, sc, row_tiles, n_tiles,
                               per_xcd, batch);
    });
}

// ---------------------------------------------------------------------------
// Row cast of a Float32 tensor (blocks along the contiguous axis; the round trip of a Float32 tensor,
// weights kept in Float32).  A wave takes 2048 consecutive elements = 64 blocks as eight fully
// coalesced 16-byte-per-lane loads (all in flight at once), parks them in a wave-private LDS region with
// a pitch of 36 dwords per block -- lane l then owns block l and reads it back with 16-byte reads that are
// free of bank conflicts (36 l mod 64 takes 16 different multiples of 4 over any 16 consecutive lanes) --
// and quantizes it with the Float32 block quantizer of the column kernel and the GEMM epilogue (hardware
// converts; the exact encoder for the rare blocks they cannot take).  No work-group barrier: waves are
// independent.  WHOLE: dense rows of whole blocks and a whole number of 2048-element runs; otherwise the
// rows are those of `geom` (see the bf16 kernel) and the last wave may have fewer than 64 blocks.
// ---------------------------------------------------------------------------
constexpr int RF_CHUNKS = 8;                       // 16-byte loads in flight per lane
constexpr int RF_WAVE_ELEMS = 64 * 4 * RF_CHUNKS;  // 2048 elements = 64 blocks per wave
constexpr int RF_PITCH = 36;                       // dwords per block in LDS

template <int FMT, int RND, bool WHOLE>
__global__ __launch_bounds__(256) void cast_row_f32_kernel(const float *__restrict__ src, RowGeom geom, uint8_t *__restrict__ elems,
                                                           uint8_t *__restrict__ scales, int64_t n_waves)
{
    if constexpr (FMT == FP8_E4M3 || FMT == FP8_E5M2) fp8_saturate_mode();
    constexpr int w = Fmt<FMT>::bits;
    __shared__ __attribute__((aligned(16))) uint32_t lds_all[4 * 64 * RF_PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t *lds = lds_all + wave * 64 * RF_PITCH;
    const int64_t wave_id = (int64_t)blockIdx.x * 4 + wave;
    if (wave_id >= n_waves) return;
    const int64_t e0 = wave_id * RF_WAVE_ELEMS, blk0 = e0 / BLOCK;

    uint4 v[RF_CHUNKS];
#pragma unroll
    for (int u = 0; u < RF_CHUNKS; u++) {
        const int64_t e = e0 + u * 256 + lane * 4;
        if constexpr (WHOLE) {
            v[u] = ld16_nt(src + e);
        } else {
            v[u] = make_uint4(0, 0, 0, 0);
            if ((e >> 2) < (int64_t)geom.n_units) {
                int n;
                const float *g = src + geom.at((uint32_t)(e >> 2), 4, n);
                if (n == 4) {
                    v[u] = ld16_nt(g);
                } else if (n > 0) {
                    uint32_t h[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) h[i] = i < n ? __float_as_uint(g[i]) : 0u;
                    v[u] = make_uint4(h[0], h[1], h[2], h[3]);
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < RF_CHUNKS; u++) {
        const int f = u * 256 + lane * 4;              // element of the wave's run: block f / 32, position f % 32
        *reinterpret_cast<uint4 *>(lds + (f >> 5) * RF_PITCH + (f & 31)) = v[u];
    }
    wave_lds_sync();
    uint32_t out[w];
    const uint32_t s = quantize_block_lds<FMT, RND>(lds + lane * RF_PITCH, 1, out);
    if (!WHOLE && blk0 + lane >= (int64_t)geom.n_units / (BLOCK / 4)) return;
    uint8_t *o = elems + (blk0 + lane) * (BLOCK * w / 8);
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
    scales[blk0 + lane] = (uint8_t)s;                  // 64 consecutive bytes per wave
}

// Dense rows of whole blocks, slices one after the other: one run of elements, counted in 64 bits
static bool one_run(const Batch &b, int64_t rows, int64_t cols, int64_t ld)
{
    return ld == cols && cols % BLOCK == 0 && (b.n == 1 || b.src == rows * ld);
}

// Other rows: their units are numbered in 31 bits, so slices of a batch, then runs of rows, go to one launch each (of 16 lines or
// blocks at a time, so that the scale bytes of a run stay 16-byte aligned).  go(batch, rows, src, lines before it);
// hipErrorNotSupported where such a run is too long.
template <typename F>
static hipError_t for_rows(const Batch &b, int64_t rows, int64_t cols, int64_t ld, int epu, int src_bytes, const void *src, F go)
{
    const int64_t nblk = (cols + BLOCK - 1) / BLOCK, most = 0x7FFFFFFF / (nblk * (BLOCK / epu));
    const char *p = static_cast<const char *>(src);
    if (b.n * rows <= most) return go(b.n, rows, p, (int64_t)0);
    const int64_t run = nblk % 16 == 0 ? most : most & ~(int64_t)15;
    if (run < 1 || (b.n > 1 && rows * nblk % 16)) return hipErrorNotSupported;
    for (int64_t i = 0; i < b.n; i++)
        for (int64_t r = 0; r < rows; r += run) {
            const hipError_t e = go((int64_t)1, rows - r < run ? rows - r : run, p + (i * b.src + r * ld) * src_bytes, i * rows + r);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

template <int FMT, int RND>
static hipError_t launch_row_f32_r(const void *src, int64_t rows, int64_t cols, int64_t ld, uint8_t *elems, uint8_t *scales, hipStream_t st,
                                   const Batch &batch)
{
    const int64_t nblk = (cols + BLOCK - 1) / BLOCK;
    auto wgs_of = [](int64_t waves) { return (waves + 3) / 4; };
    const int64_t all = batch.n * rows * nblk;
    if (one_run(batch, rows, cols, ld) && all % 64 == 0 && wgs_of(all / 64) <= 0x7FFFFFFF) {
        hipLaunchKernelGGL((cast_row_f32_kernel<FMT, RND, true>), dim3((unsigned)wgs_of(all / 64)), dim3(256), 0, st,
                           static_cast<const float *>(src), RowGeom{}, elems, scales, all / 64);
        return hipGetLastError();
    }
    return for_rows(batch, rows, cols, ld, 4, 4, src, [&](int64_t nb, int64_t nr, const char *p, int64_t line0) {
        const int64_t n_waves = (nb * nr * nblk + 63) / 64;
        const RowGeom geom = row_geom(nb, nr, cols, ld, nb > 1 ? batch.src : nr * ld, 4);
        hipLaunchKernelGGL((cast_row_f32_kernel<FMT, RND, false>), dim3((unsigned)wgs_of(n_waves)), dim3(256), 0, st,
                           reinterpret_cast<const float *>(p), geom, elems + line0 * nblk * (BLOCK * Fmt<FMT>::bits / 8),
                           scales + line0 * nblk, n_waves);
        return hipGetLastError();
    });
}

template <int FMT>
static hipError_t launch_f32_fmt(int rnd, const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems,
                                 uint8_t *scales, hipStream_t st, const Batch &batch)
{
    if (axis == 0)
        return rnd == ROUND_RNE ? launch_col_f32_r<FMT, ROUND_RNE>(src, rows, cols, ld, elems, scales, st, batch)
                                : launch_col_f32_r<FMT, ROUND_HALF_AWAY>(src, rows, cols, ld, elems, scales, st, batch);
    return rnd == ROUND_RNE ? launch_row_f32_r<FMT, ROUND_RNE>(src, rows, cols, ld, elems, scales, st, batch)
                            : launch_row_f32_r<FMT, ROUND_HALF_AWAY>(src, rows, cols, ld, elems, scales, st, batch);
}

hipError_t launch_cast_f32_fast(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, int fmt, int rnd,
                                uint8_t *elems, uint8_t *scales, hipStream_t st, const Batch &batch)
{
    switch (fmt) {
        case FP8_E4M3: return launch_f32_fmt<FP8_E4M3>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP8_E5M2: return launch_f32_fmt<FP8_E5M2>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP6_E3M2: return launch_f32_fmt<FP6_E3M2>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP6_E2M3: return launch_f32_fmt<FP6_E2M3>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP4_E2M1: return launch_f32_fmt<FP4_E2M1>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        default:       return launch_f32_fmt<INT8>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
    }
}

template <int FMT, int RND>
static hipError_t launch_fast_t(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems,
                                uint8_t *scales, hipStream_t st, const Batch &batch)
{
    if (axis == 1) {
        const int64_t pcols = (cols + BLOCK - 1) / BLOCK * BLOCK;
        auto wgs_of = [](int64_t n) { return (n + 4 * ROW_WAVE_ELEMS - 1) / (4 * ROW_WAVE_ELEMS); };
        const int64_t all = batch.n * rows * pcols;
        if (one_run(batch, rows, cols, ld) && wgs_of(all) <= 0x7FFFFFFF) {
            const uint16_t *p = static_cast<const uint16_t *>(src);
            const dim3 grid((unsigned)wgs_of(all));
            if (all % (4 * ROW_WAVE_ELEMS) == 0)
                hipLaunchKernelGGL((cast_row_bf16_kernel<FMT, RND, true, true>), grid, dim3(256), 0, st, p, RowGeom{}, elems, scales, all);
            else
                hipLaunchKernelGGL((cast_row_bf16_kernel<FMT, RND, true>), grid, dim3(256), 0, st, p, RowGeom{}, elems, scales, all);
            return hipGetLastError();
        }
        return for_rows(batch, rows, cols, ld, 8, 2, src, [&](int64_t nb, int64_t nr, const char *q, int64_t line0) {
            const int64_t n = nb * nr * pcols;
            const RowGeom geom = row_geom(nb, nr, cols, ld, nb > 1 ? batch.src : nr * ld, 8);
            hipLaunchKernelGGL((cast_row_bf16_kernel<FMT, RND, false>), dim3((unsigned)wgs_of(n)), dim3(256), 0, st,
                               reinterpret_cast<const uint16_t *>(q), geom, elems + line0 * (pcols * Fmt<FMT>::bits / 8),
                               scales + line0 * (pcols / BLOCK), n);
            return hipGetLastError();
        });
    }
    const int64_t row_tiles = (rows + COL_TILE_R - 1) / COL_TILE_R;
    // 128-column tiles once they still give every compute unit several work-groups, unless half of the last one of a few would hold
    // no columns (128 matrices of 2048 x 64 bf16, 128- / 64-column tiles, us: E4M3 18.3 / 10.6, E3M2 17.7 / 9.9; of 192
    // 39.0 / 27.4, 37.9 / 26.0; 32 of 2048 x 320 16.9 / 12.7)
    const int64_t strips = (cols + 63) / 64;
    const bool wide = (strips % 2 == 0 || strips > 16) && row_tiles * ((cols + 127) / 128) * batch.n >= 1024;
    const int64_t n_tiles = row_tiles * (wide ? (cols + 127) / 128 : (cols + 63) / 64);
    const int64_t per_xcd = (n_tiles + 7) / 8;
    if (per_xcd * 8 > 0x7FFFFFFF) return hipErrorNotSupported;
    const bool whole = rows % COL_TILE_R == 0 && cols % (wide ? 128 : 64) == 0;
#define MX_COL_GO(TC_, WHOLE_)                                                                                               \
    hipLaunchKernelGGL((cast_col_bf16_kernel<FMT, RND, TC_, WHOLE_>), grid, dim3(256), 0, st, p, rows, cols, ld, e, sc, row_tiles, n_tiles, \
                       per_xcd, batch)
    return for_batch(batch, 2, src, elems, scales, [&](unsigned nz, const char *s, uint8_t *e, uint8_t *sc) {
        const dim3 grid((unsigned)(per_xcd * 8), 1, nz);
        const uint16_t *p = reinterpret_cast<const uint16_t *>(s);
        if (wide) { if (whole) MX_COL_GO(128, true); else MX_COL_GO(128, false); }
        else      { if (whole) MX_COL_GO(64, true); else MX_COL_GO(64, false); }
    });
#undef MX_COL_GO
}

template <int FMT>
static hipError_t launch_fast_r(int rnd, const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, uint8_t *elems,
                                uint8_t *scales, hipStream_t st, const Batch &batch)
{
    return rnd == ROUND_RNE ? launch_fast_t<FMT, ROUND_RNE>(src, rows, cols, ld, axis, elems, scales, st, batch)
                            : launch_fast_t<FMT, ROUND_HALF_AWAY>(src, rows, cols, ld, axis, elems, scales, st, batch);
}

hipError_t launch_cast_bf16_fast(const void *src, int64_t rows, int64_t cols, int64_t ld, int axis, int fmt, int rnd,
                                 uint8_t *elems, uint8_t *scales, hipStream_t st, const Batch &batch)
{
    switch (fmt) {
        case FP8_E4M3: return launch_fast_r<FP8_E4M3>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP8_E5M2: return launch_fast_r<FP8_E5M2>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP6_E3M2: return launch_fast_r<FP6_E3M2>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP6_E2M3: return launch_fast_r<FP6_E2M3>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        case FP4_E2M1: return launch_fast_r<FP4_E2M1>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
        default:       return launch_fast_r<INT8>(rnd, src, rows, cols, ld, axis, elems, scales, st, batch);
    }
}

}  // namespace mx
