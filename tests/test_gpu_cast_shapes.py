"""Casts and dequantize at the edges of their kernels' tiles: strided rows, partial last blocks, row and
column remainders, batches of slices -- bit for bit against the reference."""
import numpy as np
import pytest
import torch

from gpu_util import same_floats, to_dev, to_host
from paper_2310_10537_amd import inputs

pytestmark = pytest.mark.gpu
NAMES = ("fp8_e4m3", "fp8_e5m2", "fp6_e3m2", "fp6_e2m3", "fp4_e2m1", "int8")


@pytest.fixture(scope="module")
def mx():
    from paper_2310_10537_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.lib()
    return binding


def source(rows, cols, dt, seed):
    """A [rows, cols] array whose blocks cycle through the degenerate cases along rows, heavy tails elsewhere."""
    x = inputs.student_t_f32((rows, cols), seed)
    x[: rows // 2, : cols // 32 * 32] = inputs.adversarial_f32(max(rows // 2, 1), max(cols // 32 * 32, 32), seed)[: rows // 2, : cols // 32 * 32]
    return x if dt == "f32" else inputs.f32_to_bf16_bits(x)


def strided(a, pad):
    """The array on the device as the left part of a wider tensor (rows start at multiples of 16 bytes)."""
    t = to_dev(a)
    step = 16 // t.element_size()
    ld = -(-(a.shape[1] + pad) // step) * step
    big = torch.full((a.shape[0], ld), 3.0e38, dtype=t.dtype, device="cuda")   # must never reach a block
    big[:, : a.shape[1]] = t
    return big[:, : a.shape[1]]


# rows around the 128-row tile and the 32-row block, columns around the 64- and 128-column tiles and the 8-element load
SHAPES = [(2, 1), (31, 7), (33, 65), (127, 63), (128, 64), (129, 129), (160, 200), (257, 72)]


@pytest.mark.parametrize("fmt", range(6), ids=NAMES)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("axis", [1, 0])
def test_cast_and_dequantize_at_tile_edges(mx, oracle, fmt, dt, axis):
    for n, (rows, cols) in enumerate(SHAPES):
        x = source(rows, cols, dt, seed=200 + n)
        for rnd, pad in ((0, 0), (1, 40)):
            e, s = mx.mx_quantize(strided(x, pad), axis, fmt, rnd)
            e_ref, s_ref = oracle.quantize(x, axis, fmt, rnd)
            assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, rnd, pad)
            for out_dt in (torch.float32, torch.bfloat16):
                out = torch.full((rows, -(-(cols + pad) // 8) * 8), 7.0, dtype=out_dt, device="cuda")
                mx.mx_dequantize(e, s, fmt, rows, cols, axis, out=out[:, :cols])
                want = oracle.dequantize(e_ref, s_ref, fmt, rows, cols, axis, dst_dt=int(out_dt == torch.bfloat16))
                assert same_floats(to_host(out[:, :cols]), want), (rows, cols, pad)
                assert torch.all(out[:, cols:] == 7.0), (rows, cols)


@pytest.mark.parametrize("fmt", [0, 3, 4, 5], ids=lambda f: NAMES[f])
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_batches_of_slices(mx, oracle, fmt, dt, axis):
    """Whole-tile and ragged slices, dense and with padded strides, in one call."""
    for shape in ((5, 128, 64), (3, 256, 128), (7, 45, 80), (2, 131, 96)):
        x = source(shape[0] * shape[1], shape[2], dt, seed=300 + shape[1]).reshape(shape)
        d = to_dev(x)
        big = torch.full((shape[0] + 1, shape[1] + 3, shape[2] + 16), 3.0e38, dtype=d.dtype, device="cuda")
        big[: shape[0], : shape[1], : shape[2]] = d
        e_ref, s_ref = oracle.quantize_3d(x, axis, fmt, 0, False)
        for t in (d, big[: shape[0], : shape[1], : shape[2]]):
            e, s = mx.mx_quantize_3d(t, axis, fmt)
            assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (shape, t.stride())
            back = torch.full_like(big, 7.0)
            for y in (None, back[: shape[0], : shape[1], : shape[2]]):
                y = mx.mx_dequantize_3d(e, s, fmt, shape, axis, dtype=d.dtype, out=y)
                assert same_floats(to_host(y), oracle.dequantize_3d(e_ref, s_ref, fmt, shape, axis, False, dst_dt=int(dt == "bf16"))), shape
            back[: shape[0], : shape[1], : shape[2]] = 7.0
            assert torch.all(back == 7.0)


@pytest.mark.parametrize("fmt", range(6), ids=NAMES)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("axis", [1, 0])
def test_stochastic_cast_at_tile_edges(mx, oracle, fmt, dt, axis):
    """Column counts on either side of a multiple of four (a Philox call serves four elements), degenerate blocks,
    and values that reach from the block maximum to far below the smallest grid step."""
    for n, (rows, cols) in enumerate(SHAPES + [(64, 130), (96, 127), (40, 256)]):
        x = inputs.bf16_bits_to_f32(source(rows, cols, "bf16", seed=400 + n)) if dt == "bf16" else source(rows, cols, dt, seed=400 + n)
        g = np.random.default_rng(500 + n)
        x[rows // 2:] *= np.exp2(g.integers(-24, 1, x[rows // 2:].shape)).astype(np.float32)
        x = inputs.f32_to_bf16_bits(x) if dt == "bf16" else x
        for pad, seed in ((0, 77), (24, 2 ** 63 + 5)):
            e, s = mx.mx_quantize_sr(strided(x, pad), axis, fmt, seed)
            e_ref, s_ref = oracle.quantize(x, axis, fmt, oracle.ROUND_STOCHASTIC, seed=seed)
            assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, pad)


def test_stochastic_cast_of_a_large_tensor(mx, oracle):
    """2^24 elements and more: a lane takes a whole block."""
    for shape, dt in (((4099, 4096), "bf16"), ((4096, 4102), "f32")):
        x = source(*shape, dt, seed=600)
        for fmt in (1, 2, 4, 5):
            for axis in (1, 0):
                e, s = mx.mx_quantize_sr(strided(x, 0), axis, fmt, 11)
                e_ref, s_ref = oracle.quantize(x, axis, fmt, oracle.ROUND_STOCHASTIC, seed=11)
                assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (shape, fmt, axis)


# whole 128 x 64 tiles; one and two blocks; row and column remainders of a tile; a last group of strips that is not full
@pytest.mark.parametrize("fmt", range(6), ids=NAMES)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_dual_cast_at_tile_edges(mx, oracle, fmt, dt):
    for n, (rows, cols) in enumerate([(32, 32), (64, 32), (128, 64), (160, 96), (96, 288), (256, 1216), (384, 1120)]):
        x = source(rows, cols, dt, seed=300 + n)
        for rnd, pad in ((0, 0), (1, 40)):
            for axis, (e, s) in zip((1, 0), mx.mx_quantize_dual(strided(x, pad), fmt, rnd)):
                e_ref, s_ref = oracle.quantize(x, axis, fmt, rnd)
                assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, axis, rnd, pad)


@pytest.mark.parametrize("fmt", range(6), ids=NAMES)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_blocks_of_zeros(mx, oracle, fmt, dt):
    """Blocks of zeros of either sign beside blocks with values, along both axes, inside and at the edges of tiles: the
    converts take them, and they come out as signed zeros under scale byte 0."""
    for n, (rows, cols) in enumerate([(160, 200), (128, 256), (33, 1000), (96, 64)]):
        x = inputs.student_t_f32((rows, cols), seed=700 + n)
        x[:, (cols // 3) // 32 * 32:cols // 2] = 0
        x[32:96] *= 0                                              # zeros that keep their signs
        x[rows - 1, :40] = -0.0
        x = x if dt == "f32" else inputs.f32_to_bf16_bits(x)
        for axis in (1, 0):
            for rnd in (0, 1, 2):
                e, s = mx.mx_quantize(strided(x, 0), axis, fmt, rnd)
                e_ref, s_ref = oracle.quantize(x, axis, fmt, rnd)
                assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, axis, rnd)
            e, s = mx.mx_quantize_sr(strided(x, 0), axis, fmt, 9)
            e_ref, s_ref = oracle.quantize(x, axis, fmt, oracle.ROUND_STOCHASTIC, seed=9)
            assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, axis)
        if rows % 32 == 0 and cols % 32 == 0:
            for axis, (e, s) in zip((1, 0), mx.mx_quantize_dual(strided(x, 0), fmt, 1)):
                e_ref, s_ref = oracle.quantize(x, axis, fmt, 1)
                assert np.array_equal(to_host(s), s_ref) and np.array_equal(to_host(e), e_ref), (rows, cols, axis)
