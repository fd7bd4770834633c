"""Few rows of A, where eight waves share K: at the edges of the row groups, of the 32 columns, of the waves' slices (fewer
chunks of 128 than waves, odd numbers of chunks, slices that are no multiple of four chunks) and of the cast on load."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev
from paper_2310_10537_amd import inputs
from test_gpu_gemm import check_product

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mx():
    from paper_2310_10537_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    binding.lib()
    return binding


SHAPES = [(1, 31, 128), (8, 33, 384), (9, 64, 1152), (16, 95, 2176), (17, 40, 4736), (32, 65, 5632), (5, 70, 11008)]


@pytest.mark.parametrize("M,N,K", SHAPES, ids=lambda v: str(v))
@pytest.mark.parametrize("fa,fb", [(0, 0), (1, 4), (2, 4), (3, 2), (4, 4), (4, 1)], ids=lambda v: str(v))
def test_slices_and_cast_on_load(mx, oracle, M, N, K, fa, fb):
    x = inputs.student_t_bf16((M, K), seed=M + fa)
    x[0, :32] = 0                                                  # a block of zeros
    x[M - 1, 64:96] = 0x0003                                       # a block of subnormals: the exact encoder
    ad = torch.full((M, K + 24), 3.0e38, dtype=torch.bfloat16, device="cuda")[:, :K]
    ad.copy_(to_dev(x))
    eb, sb = oracle.quantize(inputs.gaussian_f32((N, K), seed=N + fb, std=0.02), 1, fb)
    b = to_dev(eb), to_dev(sb)
    for rnd in (0, 1):
        ea, sa = oracle.quantize(x, 1, fa, rnd)
        a = to_dev(ea), to_dev(sa)
        for dt in (torch.float32, torch.bfloat16):
            C = mx.mx_gemm(*a, fa, *b, fb, K, dtype=dt)
            if dt == torch.float32 and rnd == 0:
                check_product(mx, oracle, C, ea, sa, fa, eb, sb, fb, K, f"few rows {M}x{N}x{K}")
            buf = torch.full((M, N + 9), 7.0, dtype=dt, device="cuda")
            mx.mx_gemm_qa(ad, fa, rnd, *b, fb, out=buf[:, :N])
            assert torch.equal(buf[:, :N], C) and bool((buf[:, N:] == 7.0).all()), (rnd, dt)


@pytest.mark.parametrize("fb", [0, 1, 4])
@pytest.mark.parametrize("fa", range(5))
def test_cast_on_load_of_nan_and_infinity(mx, fa, fb):
    """Non-finite values of either operand, in every chunk of a wave's slice, give what the stand-alone cast and product give."""
    K = 8192                                                       # eight chunks a wave
    for fill in (float("nan"), float("inf"), -float("inf")):
        x, w = torch.randn((16, K), device="cuda").to(torch.bfloat16), torch.randn((96, K), device="cuda")
        for c in range(K // 128):
            x[1 + c % 8, c * 128 + 40] = fill
            w[(5 * c) % 64, c * 128 + 90] = fill
        b = mx.mx_quantize(w, 1, fb)
        for rnd in (0, 1):
            want = mx.mx_gemm(*mx.mx_quantize(x, 1, fa, rnd), fa, *b, fb, K)
            got = mx.mx_gemm_qa(x, fa, rnd, *b, fb, dtype=torch.float32)
            assert torch.equal(got.isnan(), want.isnan()) and not got[0, 64:].isnan().any()
            assert torch.equal(torch.nan_to_num(got, 1.0, 2.0, 3.0), torch.nan_to_num(want, 1.0, 2.0, 3.0))


@pytest.mark.parametrize("M,N,K", [(2, 33, 2 ** 23 + 128), (130, 40, 2 ** 23 + 256), (3, 33, 2 ** 25 + 128)], ids=lambda v: str(v))
def test_k_beyond_2_23(mx, M, N, K):
    """Long K, where each wave walks an eighth: the end of the range of the other kernels, and of the staged form's 32-bit offsets."""
    g = torch.Generator(device="cuda").manual_seed(M)

    def operand(rows):
        e = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=g)
        s = torch.randint(120, 130, (rows, K // 32), dtype=torch.uint8, device="cuda", generator=g)
        return e, s

    A, B = operand(M), operand(N)
    C = mx.mx_gemm(*A, 4, *B, 4, K)
    a, b = (mx.mx_dequantize(*t, 4, r, K, 1).double() for t, r in ((A, M), (B, N)))
    want, scale = a @ b.T, a.abs() @ b.abs().T
    # Float32 sums of exact products: K / 64 additions in eight chains, errors of either sign
    assert bool(((C.double() - want).abs() <= scale * 2.0 ** -24 * (K / 512) ** 0.5 * 4).all())
