"""GPU parity at sizes past the 32-bit limits: tensors of more than 2^31 elements and more than
2^32 bytes, so that an index or a byte offset computed in 32 bits anywhere on the path lands on
the wrong bytes.  The CPU reference recomputes sampled rows, columns and entries, chosen at the
highest addresses and around the 2^31-element line."""
import numpy as np
import pytest
import torch

from paper_2310_10537_amd import inputs

pytestmark = pytest.mark.gpu

from gpu_util import same_floats, to_dev, to_host  # noqa: E402
from test_gpu_gemm import check_gemm, sampled_check  # noqa: E402

RNE = 0
PIECE_ROWS, COLS, PIECES = 2048, 65536, 20          # 40960 x 65536 = 2.68e9 elements, 5.4e9 source bytes
ROWS = PIECE_ROWS * PIECES


@pytest.fixture(scope="module")
def mx():
    from paper_2310_10537_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.lib()
    return binding


def piece_shift(p):
    return p % 7 - 3


def scaled_bits(piece_bits, k):
    """bf16 bit patterns times 2^k; exact for the N(0,1) piece (no overflow, no subnormals reached)."""
    f = (piece_bits.astype(np.uint32) << 16).view(np.float32) * np.float32(2.0 ** k)
    out = (f.view(np.uint32) >> 16).astype(np.uint16)
    assert np.array_equal((out.astype(np.uint32) << 16).view(np.float32), f)
    return out


@pytest.fixture(scope="module")
def big():
    """The big bf16 tensor: twenty copies of one seeded 2048 x 65536 N(0,1) piece, copy p scaled
    by 2^(p % 7 - 3) so that neighbouring copies differ.  Returns (host piece bits, device tensor)."""
    piece = inputs.gaussian_bf16((PIECE_ROWS, COLS), seed=900)
    pd = to_dev(piece)
    x = torch.empty((ROWS, COLS), dtype=torch.bfloat16, device="cuda")
    for p in range(PIECES):
        x[p * PIECE_ROWS:(p + 1) * PIECE_ROWS] = pd * (2.0 ** piece_shift(p))
    torch.cuda.synchronize()
    yield piece, x
    del x
    torch.cuda.empty_cache()


def host_rows(piece, r0, r1):
    out = np.empty((r1 - r0, COLS), np.uint16)
    for r in range(r0, r1):
        out[r - r0] = scaled_bits(piece[r % PIECE_ROWS], piece_shift(r // PIECE_ROWS))
    return out


def host_cols(piece, c0, c1):
    return np.concatenate([scaled_bits(piece[:, c0:c1], piece_shift(p)) for p in range(PIECES)], axis=0)


ROW_SAMPLES = [(0, 32), (32768 - 16, 32768 + 16), (ROWS - 64, ROWS)]       # row 32768 starts at element 2^31
COL_SAMPLES = [(0, 64), (30016, 30080), (COLS - 64, COLS)]


@pytest.mark.parametrize("fmt", [0, 4], ids=["fp8_e4m3", "fp4_e2m1"])
def test_cast_and_dequantize_beyond_2_31_elements(mx, oracle, big, fmt):
    piece, x = big
    bits = 8 if fmt == 0 else 4
    # blocks along the rows' own axis
    e, s = mx.mx_quantize(x, 1, fmt, RNE)
    torch.cuda.synchronize()
    assert e.shape == (ROWS, COLS * bits // 8) and s.shape == (ROWS, COLS // 32)
    y = mx.mx_dequantize(e, s, fmt, ROWS, COLS, 1, dtype=torch.bfloat16)
    for r0, r1 in ROW_SAMPLES:
        src = host_rows(piece, r0, r1)
        assert np.array_equal(to_host(x[r0:r1]), src)
        e_ref, s_ref = oracle.quantize(src, 1, fmt, RNE)
        assert np.array_equal(to_host(e[r0:r1]), e_ref), (fmt, r0)
        assert np.array_equal(to_host(s[r0:r1]), s_ref), (fmt, r0)
        y_ref = oracle.dequantize(e_ref, s_ref, fmt, r1 - r0, COLS, 1)
        assert same_floats(to_host(y[r0:r1]), inputs.f32_to_bf16_bits(y_ref)), (fmt, r0)
    del e, s, y
    # blocks along axis 0: output line c holds column c, 40960 elements long
    e, s = mx.mx_quantize(x, 0, fmt, RNE)
    torch.cuda.synchronize()
    assert e.shape == (COLS, ROWS * bits // 8) and s.shape == (COLS, ROWS // 32)
    y = mx.mx_dequantize(e, s, fmt, ROWS, COLS, 0, dtype=torch.bfloat16)      # back to [ROWS][COLS]
    assert y.shape == (ROWS, COLS)
    for c0, c1 in COL_SAMPLES:
        src = host_cols(piece, c0, c1)
        e_ref, s_ref = oracle.quantize(src, 0, fmt, RNE)
        assert np.array_equal(to_host(e[c0:c1]), e_ref), (fmt, c0)
        assert np.array_equal(to_host(s[c0:c1]), s_ref), (fmt, c0)
        y_ref = oracle.dequantize(e_ref, s_ref, fmt, ROWS, c1 - c0, 0)
        assert same_floats(to_host(y[:, c0:c1]), inputs.f32_to_bf16_bits(y_ref)), (fmt, c0)
    del e, s, y
    torch.cuda.empty_cache()


def test_dual_cast_beyond_2_31_elements(mx, oracle, big):
    piece, x = big
    (e1, s1), (e0, s0) = mx.mx_quantize_dual(x, 0, RNE)
    torch.cuda.synchronize()
    for r0, r1 in ROW_SAMPLES:
        e_ref, s_ref = oracle.quantize(host_rows(piece, r0, r1), 1, 0, RNE)
        assert np.array_equal(to_host(e1[r0:r1]), e_ref) and np.array_equal(to_host(s1[r0:r1]), s_ref)
    for c0, c1 in COL_SAMPLES:
        e_ref, s_ref = oracle.quantize(host_cols(piece, c0, c1), 0, 0, RNE)
        assert np.array_equal(to_host(e0[c0:c1]), e_ref) and np.array_equal(to_host(s0[c0:c1]), s_ref)
    del e1, s1, e0, s0
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_gemm_output_beyond_2_31_entries(mx, oracle, dt):
    """49152 x 49152 output (2.4e9 entries; 9.7e9 bytes as Float32), K = 512, on the tiled kernel."""
    M = N = 49152
    K = 512
    a = inputs.gaussian_bf16((M, K), seed=910)
    b = inputs.gaussian_bf16((N, K), seed=911)
    Ah, Bh = oracle.quantize(a, 1, 0, RNE), oracle.quantize(b, 1, 0, RNE)
    C = mx.mx_gemm(to_dev(Ah[0]), to_dev(Ah[1]), 0, to_dev(Bh[0]), to_dev(Bh[1]), 0, K, dtype=dt)
    torch.cuda.synchronize()
    assert C.shape == (M, N)
    got, C_ref, C_abs, hw = sampled_check(mx, oracle, C, Ah, 0, Bh, 0, K, seed=912)
    if dt == torch.bfloat16:
        C_abs = C_abs + np.abs(C_ref) * 2.0 ** -8 / 1e-5
    check_gemm(got, C_ref, C_abs, "large C", hw)
    # the last rows in full: every column tile of the highest row tile
    mi = np.repeat(np.arange(M - 2, M), N)
    ni = np.tile(np.arange(N), 2)
    ref, ref_abs = oracle.gemm_entries(Ah[0], Ah[1], 0, Bh[0], Bh[1], 0, K, mi, ni)
    got = C[M - 2:].float().cpu().numpy().astype(np.float64).reshape(-1)
    if dt == torch.bfloat16:
        ref_abs = ref_abs + np.abs(ref) * 2.0 ** -8 / 1e-5
    check_gemm(got, ref, ref_abs, "large C last rows", None)
    del C
    torch.cuda.empty_cache()


def test_stochastic_counter_beyond_2_32(mx, oracle):
    """286720 x 65536 bf16 (1.9e10 elements): the generator's counter, element number / 4, passes
    2^32 at row 262144, so its upper word is in use.  Blocks on both sides of that row and at the
    end are recomputed with offsets drawn per element number."""
    SR, fmt, seed = 3, 4, 0x1234567890ABCDEF
    pieces = 140
    rows = pieces * PIECE_ROWS
    piece = inputs.gaussian_bf16((PIECE_ROWS, COLS), seed=901)
    pd = to_dev(piece)
    x = torch.empty((rows, COLS), dtype=torch.bfloat16, device="cuda")
    for p in range(pieces):
        x[p * PIECE_ROWS:(p + 1) * PIECE_ROWS] = pd
    del pd
    torch.cuda.synchronize()

    def block(values, numbers):
        u = np.array([oracle.sr_uniform(seed, int(e)) for e in numbers])
        v = (values.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        sb, codes = oracle.quantize_block(v, fmt, SR, u=u)
        c = codes.astype(np.uint8)
        return sb, c[0::2] | (c[1::2] << 4)                      # FP4: two codes per byte, first in the low half

    sample_rows = (0, 262143, 262144, 262145, rows - 1)
    e, s = mx.mx_quantize_sr(x, 1, fmt, seed)
    torch.cuda.synchronize()
    eh = {r: to_host(e[r]) for r in sample_rows}
    sh = {r: to_host(s[r]) for r in sample_rows}
    del e, s
    for r in sample_rows:
        for b in (0, 1, 1000, COLS // 32 - 1):
            cols = np.arange(b * 32, b * 32 + 32)
            sb, packed = block(piece[r % PIECE_ROWS, cols], r * COLS + cols)
            assert sh[r][b] == sb, (r, b)
            assert np.array_equal(eh[r][b * 16:(b + 1) * 16], packed), (r, b)

    sample_cols = (0, 1, 40001, COLS - 1)
    e, s = mx.mx_quantize_sr(x, 0, fmt, seed)
    torch.cuda.synchronize()
    eh = {c: to_host(e[c]) for c in sample_cols}
    sh = {c: to_host(s[c]) for c in sample_cols}
    del e, s, x
    torch.cuda.empty_cache()
    for c in sample_cols:
        for rb in (0, 8191, 8192, 8193, rows // 32 - 1):
            rr = np.arange(rb * 32, rb * 32 + 32)
            sb, packed = block(piece[rr % PIECE_ROWS, c], rr * COLS + c)
            assert sh[c][rb] == sb, (c, rb)
            assert np.array_equal(eh[c][rb * 16:(rb + 1) * 16], packed), (c, rb)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_one_row_beyond_2_32_elements(mx, oracle, dt):
    """A single row of 2^32 + 72 elements (a flattened tensor with a partial last block): the columns at its end, and at
    its start, which an offset cut to 32 bits would read and write in their place."""
    fmt, cols, t0 = 0, 2 ** 32 + 72, 2 ** 32 - 64
    # rows of 4096 of one seeded piece, each scaled by its own power of two, so that no two places near the ends are alike
    piece = inputs.gaussian_f32((1, 4096), seed=920) if dt == torch.float32 else inputs.gaussian_bf16((1, 4096), seed=920)
    x = torch.empty((1, -(-cols // 4096) * 4096), dtype=dt, device="cuda")
    x.view(-1, 4096)[:] = to_dev(piece)
    x[0, :4096] *= 2
    x[0, t0:] *= 4
    x = x[:, :cols]
    e, s = mx.mx_quantize(x, 1, fmt, RNE)
    y = mx.mx_dequantize(e, s, fmt, 1, cols, 1, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for a, b in ((0, 256), (t0, cols)):
        e_ref, s_ref = oracle.quantize(to_host(x[:, a:b]), 1, fmt, RNE)
        assert np.array_equal(to_host(e[:, a:a + e_ref.shape[1]]), e_ref), (a, b)
        assert np.array_equal(to_host(s[:, a // 32:a // 32 + s_ref.shape[1]]), s_ref), (a, b)
        y_ref = oracle.dequantize(e_ref, s_ref, fmt, 1, b - a, 1, dst_dt=1)
        assert same_floats(to_host(y[:, a:b]), y_ref), (a, b)
    del x, e, s, y
    torch.cuda.empty_cache()
