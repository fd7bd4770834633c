/*
 * mx.h -- C ABI of the MI355X (gfx950) Microscaling library.
 *
 * Operations (arXiv 2310.10537):
 *   mx_quantize    Algorithm 1 (Section 3): float tensor -> MX blocks of 32
 *                  elements sharing one E8M0 power-of-two scale (Table 1).
 *   mx_quantize_dual  the same cast along both axes in one pass (Section 4.1:
 *                  a tensor and its transpose are quantized separately).
 *   mx_dequantize  v_i = X * P_i (Section 2).
 *   mx_gemm        the dot-product operation of the compute flow (Section 4.1):
 *                  both operands MX, scalar-float output.
 *   mx_gemm_qa     same with the activation operand cast on the fly
 *                  (Section 4.1, Figure 2: the cast feeds the MatMul directly).
 *
 * Conventions common to all entry points
 *   - Every tensor pointer is DEVICE memory owned by the caller; the library
 *     keeps no pointer after the call returns.  The casts and mx_dequantize
 *     never allocate.  Some GEMM routes need scratch memory: the plain entry
 *     points take it from the memory pool in stream order, the _ws forms from
 *     a caller-owned workspace (see "Scratch memory of the GEMM entry points").
 *   - hip_stream is a hipStream_t passed as void* (NULL = the default
 *     stream).  Work is enqueued on it asynchronously; no call synchronises.
 *   - The return value is an mx_status_t.  Argument errors (every status but
 *     MX_ERR_LAUNCH and a pool refusal reported as MX_ERR_WORKSPACE) are found
 *     before anything is launched: no output byte was written.  Calls that issue
 *     several launches (a ragged GEMM = interior + fringe, cast + product) can
 *     fail with MX_ERR_LAUNCH after earlier launches have written part of the
 *     output.
 *   - A zero-sized problem (rows, cols, M or N equal to 0) is MX_OK and a no-op.
 *   - Block size is 32 and the scale format is E8M0 for every element format.
 *
 * Storage of an MX tensor (the paper leaves the layout open, Section 2):
 *   two separate arrays.  For a logical [R][L] tensor blocked along L
 *   (L a multiple of 32):
 *     elems  uint8 [R][L*bits/8]  element j of a row occupies bits
 *                                 [j*bits, (j+1)*bits) of the row's byte
 *                                 string, little-endian (FP4: even element in
 *                                 the low nibble; FP6: four elements per
 *                                 three bytes);
 *     scales uint8 [R][L/32]      E8M0: X = 2^(byte-127); 0xFF = NaN.
 */
#ifndef MX_H
#define MX_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Element data formats (Table 1). */
typedef enum {
    MX_FP8_E4M3 = 0,
    MX_FP8_E5M2 = 1,
    MX_FP6_E3M2 = 2,
    MX_FP6_E2M3 = 3,
    MX_FP4_E2M1 = 4,
    MX_INT8     = 5
} mx_format_t;

/* Rounding of V/X onto the element grid: ties to even (Section 4.3) or ties
 * away from zero (Section 4.5), the two modes the paper studies.  Two more are
 * extensions of this library: the magnitude truncated (toward zero), and
 * stochastic rounding -- the magnitude goes to the next grid value up with
 * probability equal to the discarded fraction of a grid step, else down -- which
 * needs a seed and therefore its own entry point, mx_quantize_sr. */
typedef enum {
    MX_ROUND_RNE = 0,
    MX_ROUND_HALF_AWAY = 1,
    MX_ROUND_TOWARD_ZERO = 2,
    MX_ROUND_STOCHASTIC = 3
} mx_round_t;

/* Scalar float types. */
typedef enum { MX_DT_F32 = 0, MX_DT_BF16 = 1 } mx_dtype_t;

typedef enum {
    MX_OK = 0,
    MX_ERR_NULL = 1,        /* a required pointer is NULL                        */
    MX_ERR_ENUM = 2,        /* format / rounding / dtype / axis out of range     */
    MX_ERR_SHAPE = 3,       /* negative size, leading dimension smaller than the
                               row length, block axis not a multiple of 32
                               where whole blocks are required (GEMM K, dual cast) */
    MX_ERR_ALIGN = 4,       /* pointer or leading dimension not 16-byte aligned  */
    MX_ERR_UNSUPPORTED = 5, /* MX_INT8 paired with another format in a GEMM      */
    MX_ERR_LAUNCH = 6,      /* the HIP runtime refused the launch                */
    MX_ERR_TOO_LARGE = 7,   /* mx_gemm_qa_noalloc: the static scratch is too small */
    MX_ERR_WORKSPACE = 8    /* a GEMM route could not get its scratch memory: caller
                               workspace too small, or the memory pool refused      */
} mx_status_t;

/* Size in bytes of the elems array for a [rows, cols] source cast along axis:
 * lines * ceil(L/32) * 32*bits/8 with L the block-axis length. */
size_t mx_elem_bytes(mx_format_t fmt, int64_t rows, int64_t cols, int axis);
/* Size in bytes of the scales array: lines * ceil(L/32). */
size_t mx_scale_bytes(int64_t rows, int64_t cols, int axis);

/*
 * Algorithm 1 over a row-major [rows, cols] tensor (Section 3).
 *   src        device, src_dt elements, row r starts at src + r*ld elements;
 *              16-byte aligned, ld*sizeof(element) a multiple of 16
 *   axis       1: blocks run along the last (contiguous) dimension;
 *                 elems [rows][cols*bits/8], scales [rows][cols/32]
 *              0: blocks run along dimension 0 and the result is stored as the
 *                 cast of the transpose, so the block axis is contiguous again:
 *                 elems [cols][rows*bits/8], scales [cols][rows/32]
 *              (the two differ: cast and transpose do not commute, Section 3)
 *   fmt, rnd   element format and rounding mode (MX_ROUND_STOCHASTIC is
 *              MX_ERR_ENUM here: see mx_quantize_sr)
 *   elems_out  device, mx_elem_bytes() bytes, 16-byte aligned
 *   scales_out device, mx_scale_bytes() bytes, 16-byte aligned
 * The block axis may have any length L.  The paper defines the cast on whole
 * blocks only; here a partial last block is filled up with zeros (they neither
 * move the block maximum nor give a non-zero code) and every stored line holds
 * ceil(L/32) whole blocks: elems [..][ceil(L/32)*32*bits/8], scales
 * [..][ceil(L/32)], which is what mx_elem_bytes / mx_scale_bytes return.  Such
 * a tensor is a valid mx_gemm operand with K = 32*ceil(L/32): the fill adds 0.
 * Per block: scale byte = clamp(floor(log2 max|V|) - emax_elem + 127, 0, 254)
 * over the normal finite inputs (0 if there are none); Float32-subnormal inputs
 * give P = 0; finite values beyond the largest normal clamp to it with their
 * sign; Inf/NaN are never clamped: they become the element Inf/NaN where the
 * format has one (FP8 E4M3 has no Inf: NaN), otherwise the whole block is
 * marked NaN by scale byte 0xFF with all element codes 0.
 */
int mx_quantize(const void *src, mx_dtype_t src_dt, int64_t rows, int64_t cols,
                int64_t ld, int axis, mx_format_t fmt, mx_round_t rnd,
                void *elems_out, uint8_t *scales_out, void *hip_stream);

/*
 * Algorithm 1 with stochastic rounding in quantize_to_element_format (an
 * extension; Section 3 leaves the element rounding to the implementation and
 * the paper's studies use the two nearest modes).  Arguments, layouts, scale
 * bytes, clamping and Inf/NaN handling as mx_quantize.  With step the grid
 * spacing of the element format at |V/X|, the stored magnitude is
 *     step * floor(|V/X| / step + u),   u = r / 2^25,
 * r the top 25 bits of word (e mod 4) of Philox4x32-10 (Salmon et al., SC 2011)
 * with key = seed and counter = e / 4, where e = row*cols + col numbers the
 * elements of the SOURCE tensor.  The offset therefore belongs to the tensor
 * element: casts of one tensor along axis 1 and axis 0 with one seed draw the
 * same u for an element, and a result can be reproduced anywhere from
 * (seed, shape).  Use a fresh seed per tensor and per step.
 */
int mx_quantize_sr(const void *src, mx_dtype_t src_dt, int64_t rows, int64_t cols,
                   int64_t ld, int axis, mx_format_t fmt, uint64_t seed,
                   void *elems_out, uint8_t *scales_out, void *hip_stream);

/*
 * Both casts of one tensor in a single call: (elems_axis1, scales_axis1) receive
 * exactly what mx_quantize writes with axis = 1 and (elems_axis0, scales_axis0)
 * what it writes with axis = 0.  A training step needs each tensor with its
 * blocks along the reduction axis of every GEMM that uses it (X and X^T, W and
 * W^T, dY and dY^T -- Section 4.1, Figure 2 -- and the two casts differ), so the
 * source is read once instead of twice.  rows and cols must both be multiples
 * of 32.  bf16 sources made of whole 128 x 64 tiles, rounded to nearest, take
 * the one-pass kernel; anything else runs the two casts one after the other.
 * Arguments, alignment and error behaviour as for mx_quantize (for stochastic
 * rounding call mx_quantize_sr twice with one seed: both axes then draw the
 * same offset for an element).
 */
int mx_quantize_dual(const void *src, mx_dtype_t src_dt, int64_t rows, int64_t cols,
                     int64_t ld, mx_format_t fmt, mx_round_t rnd,
                     void *elems_axis1, uint8_t *scales_axis1,
                     void *elems_axis0, uint8_t *scales_axis0, void *hip_stream);

/*
 * Algorithm 1 along any axis of a 3-D tensor (Section 3: each tensor has a
 * principal axis along which its blocks run; for a multi-dimensional tensor
 * that can be any of its axes).  src holds [d0][d1][d2] with element (i0, i1,
 * i2) at src + i0*stride0 + i1*stride1 + i2 (strides in elements, the last
 * axis contiguous, stride1 >= d2, stride0 >= d1*stride1; src 16-byte aligned
 * and both strides a multiple of 16 bytes) -- a batch of matrices, a slice of
 * a larger tensor, or with d0 = 1 a plain matrix.  axis = 0, 1 or 2 names the
 * block axis, of length L.  Two output layouts:
 *   keep_order = 0  the block axis is moved last and the other two keep their
 *       order, i.e. the 2-D cast of the permuted tensor: with (o1, o2) the two
 *       remaining indices,  elems [o1][o2][ceil(L/32)*32*bits/8],
 *       scales [o1][o2][ceil(L/32)].  Each [o1] slice is what mx_quantize writes
 *       for the matching 2-D problem (axis = 2: rows of the slice; axis = 1:
 *       its axis-0 cast), so a slice is a valid mx_gemm operand.
 *   keep_order = 1  the untransposed form: codes stay at their element's place,
 *       packed along the last axis (d2*bits must be a multiple of 8):
 *       elems [d0][d1][d2*bits/8]; scales has the source's shape with the block
 *       axis replaced by its block count: [d0][d1][ceil(d2/32)],
 *       [d0][ceil(d1/32)][d2] or [ceil(d0/32)][d1][d2].  A partial last block
 *       is cast as if filled up with zeros; nothing is stored for the fill.
 * rnd: not MX_ROUND_STOCHASTIC.  Outputs 16-byte aligned device memory.
 * Slices go through one launch (one per 65535 of them)
 * (MX_ERR_UNSUPPORTED beyond 65535 * 32 rows along the block axis with
 * keep_order = 1).
 */
int mx_quantize_3d(const void *src, mx_dtype_t src_dt,
                   int64_t d0, int64_t d1, int64_t d2, int64_t stride0, int64_t stride1,
                   int axis, mx_format_t fmt, mx_round_t rnd, int keep_order,
                   void *elems_out, uint8_t *scales_out, void *hip_stream);

/*
 * Inverse of mx_quantize_3d (Section 2: v_i = X * P_i): elems / scales in either
 * of its layouts (keep_order as there; axis names the block axis) back to a
 * [d0][d1][d2] tensor of type dst_dt written at dst[i0*stride0 + i1*stride1 + i2]
 * (elements; stride1 >= d2, stride0 >= d1*stride1, dst 16-byte aligned and both
 * strides a multiple of 16 bytes).  Nothing outside the tensor's elements is
 * written.  A scale byte 0xFF gives NaN for its block; fill positions of a
 * partial last block (keep_order = 0) are skipped.
 */
int mx_dequantize_3d(const void *elems, const uint8_t *scales, mx_format_t fmt,
                     int64_t d0, int64_t d1, int64_t d2, int axis, int keep_order,
                     void *dst, mx_dtype_t dst_dt, int64_t stride0, int64_t stride1,
                     void *hip_stream);

/*
 * v = X * P (Section 2) for an MX tensor produced by mx_quantize with the same
 * rows, cols and axis; writes row-major dst [rows, cols] with leading
 * dimension ld (elements).  Scale byte 0xFF gives NaN for the whole block;
 * |X*P| beyond Float32 range gives +-Inf.  Pointers 16-byte aligned.  With a
 * block-axis length that is not a multiple of 32 the fill positions of the
 * last block are skipped.
 */
int mx_dequantize(const void *elems, const uint8_t *scales, mx_format_t fmt,
                  int64_t rows, int64_t cols, int axis,
                  void *dst, mx_dtype_t dst_dt, int64_t ld, void *hip_stream);

/*
 * MX dot products (Section 4.1):
 *   C[m][n] = sum over blocks b of X_A[m][b] * X_B[n][b] * sum_j a[m][32b+j] * b[n][32b+j]
 * A is an MX tensor [M][K] and B an MX tensor [N][K], both blocked along K as
 * written by mx_quantize (axis = 1, or axis = 0 of the transposed source);
 * K must be a multiple of 32.  The products go through gfx950's block-scaled
 * matrix instruction and are accumulated in Float32; that instruction adds each
 * run of 8 consecutive K products in fixed point with 14 bits below the run's
 * largest product, which is exact for FP6 E2M3 / FP4 E2M1 operands and loses at
 * most 14 * 2^-14 of each run's largest product otherwise.
 * Which kernel runs depends on the shape and the formats only, never on
 * timing or (MXINT8 near the end of Float32's range apart, see below) on the data,
 * so a result is reproducible.  Most problems add the
 * products of an entry in the order of K: whole 256 x 256 tiles (K a multiple of
 * 128), smaller tiles for every other size, and one wave per 32 x 32 entries for
 * a short K, all with the same bits.  Problems of few rows (up to 32; up to 64
 * where N is small), small ones (fewer than 24 tiles of 64 x 64, K below 4096)
 * and those with K beyond 2^23 split K over the eight waves of a work-group
 * instead and add the eight partial sums in a fixed order: a different Float32
 * rounding.
 * C is row-major [M][N] of type c_dt with leading dimension ldc >= N (elements;
 * any value, a multiple of 16 bytes is fastest); the C pointer is 16-byte
 * aligned; bf16 output is the Float32 accumulator rounded to nearest even.
 * fmtA / fmtB may differ, except that MX_INT8 pairs only with MX_INT8 (anything
 * else is MX_ERR_UNSUPPORTED).  That pair runs the integer matrix instruction
 * block by block -- every block sum is an exact integer -- and adds the scaled
 * block sums in Float32; larger problems (whole 256 x 256 tiles, at least 96 or 64
 * when K < 1024; other sizes of more than 128 rows that the integer kernels take
 * about 100 us for, see mx_gemm_workspace_bytes) instead write the elements times
 * their scales as bf16 numbers, which hold them exactly, to scratch memory
 * ((M + N) * K * 2 bytes and some, see "Scratch memory of the GEMM entry points" below)
 * and run a bf16 product with Float32 sums; 64 x 64 tiles of C whose scale bytes
 * are so large that a sum could overflow (two bytes that add up to more than
 * 379 - log2 K: products beyond 2^(127 - log2 K)) are recomputed block by block,
 * the one place where data has a say in how an entry is computed; few rows (M <= 128, K >= 256) and mid-size
 * problems with a long K let eight waves share the K range of each 32-column
 * tile and add their partial tiles in a fixed order.  All routes differ from
 * the exact sum only by Float32 accumulation rounding.
 */
int mx_gemm(int64_t M, int64_t N, int64_t K,
            const void *A_elems, const uint8_t *A_scales, mx_format_t fmtA,
            const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
            void *C, mx_dtype_t c_dt, int64_t ldc, void *hip_stream);

/*
 * Same product with A given as raw bf16 [M][K] (leading dimension lda
 * elements, a multiple of 8) and cast to fmtA with rounding rnd while it is
 * loaded.  The result is bit-identical to mx_quantize(A, axis 1) followed by
 * mx_gemm.
 * The routes, chosen by shape:
 *   - up to 16 rows with K a multiple of 128 that mx_gemm gives to its kernel for
 *     few rows: cast by that kernel (no scratch);
 *   - 8-bit formats on whole 256 x 256 tiles, at most two columns and at least 256
 *     of them: cast in the K loop of the tiled kernel (no scratch; a fringe of rows
 *     or columns beside the tiles is a product of its own and may need some);
 *   - more than 128 rows and a K below 512 or no multiple of 128: cast in registers
 *     (no scratch) where that is faster, otherwise as the rest; and in registers
 *     too when scratch memory is refused, so such a call never fails for want of it;
 *   - the rest: A is cast into scratch memory of M*K*(bits/8 + 1/32) bytes first
 *     (MX_INT8 too, whose large products take scratch of their own, see mx_gemm).
 * The casts without scratch round to nearest: MX_ROUND_TOWARD_ZERO always casts
 * into scratch first; MX_ROUND_STOCHASTIC is
 * MX_ERR_ENUM.  Where the scratch comes from, and what happens when there is
 * none, is stated under "Scratch memory of the GEMM entry points" below.
 */
int mx_gemm_qa(int64_t M, int64_t N, int64_t K,
               const void *A_bf16, int64_t lda, mx_format_t fmtA, mx_round_t rnd,
               const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
               void *C, mx_dtype_t c_dt, int64_t ldc, void *hip_stream);

/*
 * Scratch memory of the GEMM entry points.  Some routes need device scratch:
 *   mx_gemm     larger MX_INT8 problems (the bf16 values of both operands; see
 *               there);
 *   mx_gemm_qa  every route that casts A ahead of the product (see there);
 *   mx_gemm_q   every route that does not cast in the tiled kernel's epilogue
 *               (a Float32 C).
 * mx_gemm / mx_gemm_qa / mx_gemm_q take it from the device's default memory
 * pool in stream order (hipMallocAsync / hipFreeAsync on hip_stream).  The _ws
 * forms below take it from the CALLER instead: `workspace` is device memory of
 * at least mx_*_workspace_bytes(...) bytes (an upper bound over the routes the
 * shape can take; 0 means the call never needs scratch), 16-byte aligned, owned
 * by the caller, and in use until the call's work on hip_stream has finished.
 * With a non-NULL workspace the library allocates nothing at all; a workspace
 * smaller than the bound is MX_ERR_WORKSPACE and nothing is launched.
 * workspace = NULL makes a _ws form behave exactly like the plain one.
 * In either form a request that cannot be met is an error (MX_ERR_WORKSPACE),
 * with two exceptions: where mx_gemm_qa can cast in registers instead (see there),
 * and where the memory pool has no room for an MX_INT8 product of other sizes than
 * whole 256 x 256 tiles, which then runs on the integer kernels (a different Float32
 * rounding).  Otherwise results are bit-identical between the two forms.  A call
 * captured into a graph without a workspace puts the allocation into the graph.
 */
size_t mx_gemm_workspace_bytes(int64_t M, int64_t N, int64_t K, mx_format_t fmtA, mx_format_t fmtB);
size_t mx_gemm_qa_workspace_bytes(int64_t M, int64_t N, int64_t K, mx_format_t fmtA, mx_format_t fmtB);
size_t mx_gemm_q_workspace_bytes(int64_t M, int64_t N, int64_t K, mx_format_t fmtA, mx_format_t fmtB);
int mx_gemm_ws(int64_t M, int64_t N, int64_t K,
               const void *A_elems, const uint8_t *A_scales, mx_format_t fmtA,
               const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
               void *C, mx_dtype_t c_dt, int64_t ldc,
               void *workspace, size_t workspace_bytes, void *hip_stream);
int mx_gemm_qa_ws(int64_t M, int64_t N, int64_t K,
                  const void *A_bf16, int64_t lda, mx_format_t fmtA, mx_round_t rnd,
                  const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
                  void *C, mx_dtype_t c_dt, int64_t ldc,
                  void *workspace, size_t workspace_bytes, void *hip_stream);
int mx_gemm_q_ws(int64_t M, int64_t N, int64_t K,
                 const void *A_elems, const uint8_t *A_scales, mx_format_t fmtA,
                 const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
                 mx_format_t fmtC, mx_round_t rnd,
                 void *C_elems, uint8_t *C_scales,
                 void *workspace, size_t workspace_bytes, void *hip_stream);

/*
 * mx_gemm_qa for callers that cannot allocate device memory: code under HIP graph
 * capture, tight serving loops, harnesses that forbid hipMalloc.  Same arguments
 * and the same result, bit for bit, as mx_gemm_qa; the difference is where the MX
 * form of A lives between the cast and the product: in a static device array of
 * MX_NOALLOC_SCRATCH_BYTES bytes inside the library (one copy per GPU, held until
 * the process ends) instead of a workspace from the memory pool.  The call makes
 * no hipMalloc / hipFree / pool request of any kind; it launches the row cast of A
 * into that array and then the kernel mx_gemm would pick for the shape.
 *   - M * K * bits(fmtA) / 8 (rounded up to 256) + M * K / 32 bytes must fit in
 *     MX_NOALLOC_SCRATCH_BYTES (36 MiB: an 8192 x 4096 8-bit operand fits);
 *     otherwise MX_ERR_TOO_LARGE and nothing is launched.
 *   - MX_INT8 operands are MX_ERR_UNSUPPORTED here (their kernels use pool
 *     workspaces of their own); rnd may be any mode mx_gemm_qa takes.
 *   - Every call on a GPU uses that GPU's one array: calls that overlap in time on
 *     one GPU (different streams, or different host threads) race on it.  Calls on
 *     one stream are ordered and safe.  Nothing in the array has to be cleared:
 *     each call overwrites the part it reads.
 *   - The array's address is looked up on the first call on a device
 *     (hipGetSymbolAddress: no allocation); make that first call outside a graph
 *     capture.
 */
#define MX_NOALLOC_SCRATCH_BYTES (36u << 20)
int mx_gemm_qa_noalloc(int64_t M, int64_t N, int64_t K,
                       const void *A_bf16, int64_t lda, mx_format_t fmtA, mx_round_t rnd,
                       const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
                       void *C, mx_dtype_t c_dt, int64_t ldc, void *hip_stream);

/*
 * The product of mx_gemm with C delivered as an MX tensor: Algorithm 1 (Section
 * 3) applied to the Float32 result along N, which is how the output of one
 * MatMul reaches the next as an operand (Figure 2).  C_elems [M][ceil(N/32)*
 * 32*bits/8] and C_scales [M][ceil(N/32)] receive, bit for bit, what
 * mx_quantize(axis 1, fmtC, rnd) writes for the Float32 C of mx_gemm.
 * Problems the LDS-tiled kernel takes (whole 256 x 256 tiles, FP8 / FP6 / FP4
 * operands, K a multiple of 128, at least 512) with a round-to-nearest mode
 * cast the accumulators in that kernel's epilogue, for every fmtC: C
 * never exists in memory at more than fmtC's width.  Everything else computes
 * C as Float32 into scratch memory (M*N*4 bytes, see "Scratch memory of the GEMM
 * entry points") and casts it.  rnd: not MX_ROUND_STOCHASTIC.  Pointers 16-byte
 * aligned, device memory, caller-owned; errors as mx_gemm.
 */
int mx_gemm_q(int64_t M, int64_t N, int64_t K,
              const void *A_elems, const uint8_t *A_scales, mx_format_t fmtA,
              const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
              mx_format_t fmtC, mx_round_t rnd,
              void *C_elems, uint8_t *C_scales, void *hip_stream);

/*
 * Measurement aid (no part of the MX path): moves bytes in the access pattern of
 * the row cast -- consecutive 16-byte pieces per lane, several loads in flight,
 * 16-byte stores -- with no arithmetic, so that a benchmark can state what that
 * pattern reaches on the box it runs on.  Reads read_per_write * dst_bytes bytes
 * from src (read_per_write = 0, 1, 2 or 4) and, if write is non-zero, writes
 * dst_bytes bytes to dst; with write = 0 the loads are kept alive by a store
 * that never happens (dst must still be a valid 16-byte buffer).  dst_bytes is
 * a multiple of 8192; pointers are 16-byte aligned device memory.
 */
int mx_stream_pattern(const void *src, void *dst, int64_t dst_bytes,
                      int read_per_write, int write, void *hip_stream);

/*
 * Measurement aid (no part of the MX path): mx_gemm's LDS-tiled kernel for one of
 * three format pairs -- E4M3 x E4M3, E3M2 x E3M2, E3M2 x E2M1 (anything else is
 * MX_ERR_UNSUPPORTED) -- with bf16 output, which also has every work-group
 * record how long it ran from its start to the end of its K loop: shader clocks
 * at probe[2*g] and ticks of the constant 100 MHz counter at probe[2*g + 1], g
 * the work-group's index in launch order.  From the two a benchmark gets the
 * shader clock under this load and the clocks per K step.  M and N are
 * multiples of 256, K a multiple of 128 and at least 512 (else MX_ERR_SHAPE);
 * probe holds probe_len >= 2 * (tiles rounded up to a multiple of 8) entries of
 * device memory, which the caller clears first (work-groups without a tile write
 * nothing).  C receives the same bytes as from mx_gemm.
 */
int mx_gemm_probe(int64_t M, int64_t N, int64_t K,
                  const void *A_elems, const uint8_t *A_scales, mx_format_t fmtA,
                  const void *B_elems, const uint8_t *B_scales, mx_format_t fmtB,
                  void *C_bf16, int64_t ldc,
                  uint64_t *probe, int64_t probe_len, void *hip_stream);

/*
 * Measurement aid (no part of the MX path): the matrix instruction of mx_gemm's
 * kernels on its own.  MX_MFMA_STREAM_WGS work-groups of four waves (one per
 * compute unit) each issue 16 * iters scaled 32 x 32 x 64 instructions of the
 * pair fmt x fmt (an FP8 / FP6 / FP4 format, else MX_ERR_UNSUPPORTED) on operand
 * registers loaded once from `codes` -- 65536 bytes of device memory, 32-byte
 * aligned: eight fragments of 256 lanes x 32 bytes, of which the narrower formats
 * use the first 24 / 16 -- with unit scales and 256 accumulator registers per
 * lane, and touch no memory inside the loop: what the instruction sustains on
 * these operand values under the chip's power limit, whatever feeds it.  A launch
 * performs MX_MFMA_STREAM_WGS * 4 * 16 * iters * 131072 flops.  Every work-group
 * writes (shader clocks, ticks of the constant 100 MHz counter) to probe[2*g],
 * probe[2*g + 1] (2 * MX_MFMA_STREAM_WGS entries) and each lane a checksum to
 * sink (MX_MFMA_STREAM_WGS * 256 floats); iters in [1, 2^20] (else MX_ERR_SHAPE).
 */
#define MX_MFMA_STREAM_WGS 256
int mx_mfma_stream_probe(mx_format_t fmt, const void *codes, int iters,
                         float *sink, uint64_t *probe, void *hip_stream);

/* Static, human-readable text for a status code. */
const char *mx_strerror(int status);

#ifdef __cplusplus
}
#endif
#endif
