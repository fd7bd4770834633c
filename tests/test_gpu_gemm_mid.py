"""The LDS-tiled kernel for problems that 256 x 256 tiles do not fit, at the edges of its tiles and of its K steps:
every output entry is one chain of the matrix instruction in increasing K, so sampled entries and the whole last row
and column must equal the instruction model bit for bit (tests/mfma_model.py)."""
import numpy as np
import pytest
import torch

import mfma_model as hw
from gpu_util import to_dev, to_host
from paper_2310_10537_amd import inputs
from test_gpu_gemm_model import NAMES, assert_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mx():
    from paper_2310_10537_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.lib()
    return binding


# 64 x 64, 64 x 128 and 128 x 128 tiles, one round and more; K below one step, whole steps with whole and partial
# scale groups, and every length of the last, partial step
SHAPES = [(129, 900, 32), (65, 1537, 96), (160, 577, 640), (127, 1601, 1024), (200, 1100, 2080), (130, 8300, 992), (300, 9001, 544),
          (600, 9000, 416)]


@pytest.mark.parametrize("M,N,K", SHAPES, ids=lambda v: str(v))
@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 3), (2, 2), (3, 4), (4, 4), (4, 1)], ids=lambda v: str(v))
def test_matches_model(mx, oracle, M, N, K, fa, fb):
    a = inputs.student_t_f32((M, K), seed=M + fa)
    b = inputs.gaussian_f32((N, K), seed=N + fb, std=0.02)
    ea, sa = oracle.quantize(a, 1, fa)
    eb, sb = oracle.quantize(b, 1, fb)
    dev = [to_dev(t) for t in (ea, sa, eb, sb)]
    Cd = mx.mx_gemm(dev[0], dev[1], fa, dev[2], dev[3], fb, K)
    rng = np.random.default_rng(5)
    mi = np.concatenate([rng.integers(0, M, 3000), np.full(64, M - 1), rng.integers(0, M, 64)])
    ni = np.concatenate([rng.integers(0, N, 3000), rng.integers(0, N, 64), np.full(64, N - 1)])
    want = hw.gemm_entries(ea, sa, fa, eb, sb, fb, K, mi, ni)
    assert_bits(to_host(Cd)[mi, ni], want, f"{NAMES[fa]} x {NAMES[fb]} {M}x{N}x{K}")
    for dt, pad in ((torch.float32, -N % 4), (torch.bfloat16, -N % 8), (torch.bfloat16, -N % 8 + 3)):   # wide and single stores
        buf = torch.full((M, N + pad), 7.0, dtype=dt, device="cuda")
        mx.mx_gemm(dev[0], dev[1], fa, dev[2], dev[3], fb, K, out=buf[:, :N])
        assert torch.equal(buf[:, :N], Cd.to(dt)), (dt, pad)
        assert pad == 0 or bool((buf[:, N:] == 7.0).all())


# one and two blocks of K, partial steps, fewer and more than a tile's rows and columns; a long odd K whose scratch is refused
@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 3), (2, 4), (3, 2), (4, 1)], ids=lambda v: str(v))
def test_cast_in_registers(mx, fa, fb):
    """Short K of many rows is cast without scratch memory: the same bits as the cast and the product apart."""
    for M, N, K in ((129, 65, 32), (300, 500, 96), (257, 64, 160), (700, 130, 128)):
        x = inputs.student_t_bf16((M, K), seed=M + fa)
        x[0, :32] = 0
        x[M - 1, K - 32:] = 0x0003                                 # a block of subnormals
        x[1, 3], x[2, K - 1] = 0x7F80, 0x7FC1                      # infinity, NaN
        a = torch.full((M, K + 24), 3.0e38, dtype=torch.bfloat16, device="cuda")[:, :K]
        a.copy_(to_dev(x))
        b = mx.mx_quantize(to_dev(inputs.gaussian_f32((N, K), seed=N + fb, std=0.02)), 1, fb)
        for rnd in (0, 1):
            ma = mx.mx_quantize(a, 1, fa, rnd)
            for dt in (torch.float32, torch.bfloat16):
                want = mx.mx_gemm(*ma, fa, *b, fb, K, dtype=dt)
                buf = torch.full((M, N + 9), 7.0, dtype=dt, device="cuda")
                mx.mx_gemm_qa_ws(a, fa, rnd, *b, fb, None, out=buf[:, :N])
                got = buf[:, :N]
                assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.nan_to_num(1.0, 2.0, 3.0), want.nan_to_num(1.0, 2.0, 3.0))
                assert bool((buf[:, N:] == 7.0).all()), (M, N, K)
