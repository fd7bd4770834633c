"""The 256 x 256 tiles and their half-width form, which take whole-tile products of more than 64 tiles, and products cut into an
interior of more than 192 whole tiles and a fringe: every format pair, plain and cast on load (tests/test_launches.py checks
without a GPU that these shapes reach the kernels they are meant for)."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev, to_host
from paper_2310_10537_amd import inputs
from test_gpu_gemm import AWAY, NAMES, RNE, check_product

pytestmark = pytest.mark.gpu

HALF = [(2816, 1792, 512), (1280, 3328, 896)]                  # 77 and 65 tiles; a whole and a partial last scale group
WHOLE = [(3072, 3072, 512), (2304, 3840, 1152)]                # 144 and 135 tiles
INTERIOR = [(3600, 3700, 512), (3600, 3584, 640), (3584, 3700, 512)]      # 196 whole tiles and both fringes, one of rows, one of columns
NARROW = (32800, 512, 512)                                      # 256 tiles cast on load by the tiled kernel, and a fringe of rows


@pytest.fixture(scope="module")
def mx():
    from paper_2310_10537_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def source(mx):
    """bf16 activations and weights whose blocks get very different scales, so that a scale byte read for the wrong row, block or
    K step shows up."""
    def make(rows, K, seed):
        x = inputs.student_t_f32((512, K), seed=seed)
        g = np.random.default_rng(seed)
        t = to_dev(np.tile(x, (-(-rows // 512), 1))[:rows])
        return (t * to_dev(np.exp2(g.integers(-6, 6, (rows, K // 32))).astype(np.float32)).repeat_interleave(32, dim=1)).to(torch.bfloat16)
    return make


def product(mx, oracle, source, shape, fa, fb, dt, seed):
    M, N, K = shape
    a, b = source(M, K, seed), source(N, K, seed + 1)
    A, B = mx.mx_quantize(a, 1, fa), mx.mx_quantize(b, 1, fb)
    C = mx.mx_gemm(*A, fa, *B, fb, K, dtype=dt)
    check_product(mx, oracle, C, to_host(A[0]), to_host(A[1]), fa, to_host(B[0]), to_host(B[1]), fb, K, f"{NAMES[fa]}x{NAMES[fb]} {shape}", seed=seed)
    return a, A, B, C


@pytest.mark.parametrize("fa", range(5), ids=NAMES)
@pytest.mark.parametrize("fb", range(5), ids=NAMES)
def test_every_pair_on_half_and_whole_tiles(mx, oracle, source, fa, fb):
    for n, shape in enumerate(HALF + WHOLE):
        dt = (torch.float32, torch.bfloat16)[(n + fa + fb) % 2]
        _, A, B, C = product(mx, oracle, source, shape, fa, fb, dt, 40 * fa + 8 * fb + n)
        pad = 2 if dt == torch.float32 else 6                  # a row pitch that rules out the wide stores
        buf = torch.full((shape[0], shape[1] + pad), 7.0, dtype=dt, device="cuda")
        mx.mx_gemm(*A, fa, *B, fb, shape[2], out=buf[:, :shape[1]])
        assert torch.equal(buf[:, :shape[1]], C) and bool((buf[:, shape[1]:] == 7.0).all()), shape


@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 1), (2, 2), (2, 4), (4, 0), (0, 3)], ids=lambda v: str(v))
def test_interior_and_fringe(mx, oracle, source, fa, fb):
    for n, shape in enumerate(INTERIOR):
        a, A, B, C = product(mx, oracle, source, shape, fa, fb, torch.float32, 300 + 10 * fa + fb + n)
        # the fringe is a product of its own rows and columns
        M, N, K = shape
        r, c = M // 256 * 256, N // 256 * 256
        for rows, cols in ((slice(r, M), slice(0, N)), (slice(0, r), slice(c, N))):
            if rows.stop > rows.start and cols.stop > cols.start:
                part = mx.mx_gemm(A[0][rows], A[1][rows], fa, B[0][cols], B[1][cols], fb, K)
                assert torch.equal(part, C[rows, cols]), (shape, rows, cols)
        out = torch.full((M, N + 4), 7.0, device="cuda")
        mx.mx_gemm_qa(a, fa, RNE, *B, fb, out=out[:, :N])
        assert torch.equal(out[:, :N], C) and bool((out[:, N:] == 7.0).all()), shape


@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 0), (2, 4)], ids=lambda v: str(v))
def test_cast_on_load_of_many_rows_with_a_fringe(mx, oracle, source, fa, fb):
    M, N, K = NARROW
    a, A, B, C = product(mx, oracle, source, NARROW, fa, fb, torch.bfloat16, 400 + fa)
    assert torch.equal(mx.mx_gemm_qa(a, fa, RNE, *B, fb, dtype=torch.bfloat16), C)
    away = mx.mx_gemm(*mx.mx_quantize(a, 1, fa, AWAY), fa, *B, fb, K, dtype=torch.bfloat16)
    assert torch.equal(mx.mx_gemm_qa(a, fa, AWAY, *B, fb, dtype=torch.bfloat16), away)
