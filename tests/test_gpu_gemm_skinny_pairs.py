"""Up to 16 rows of A: the widths of its loads (8, 16 or 32 rows; against 4-bit weights two chunks at a time).  Each entry's products are
added in the order of the 32-row form, so the rows of a 17-row product are the same bits; the 32-row form is held to the oracle elsewhere.
Chunks per wave: one, an odd number, the last wave of fewer -- the second chunk of a pair then lies beyond the slice or beyond K."""
import pytest
import torch

FORMATS = [(0, 4), (2, 4), (4, 4), (0, 0), (2, 3), (4, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("K", [128, 384, 1408, 3072, 4224], ids=lambda k: f"chunks{k // 128}")
@pytest.mark.parametrize("fa,fb", FORMATS, ids=lambda f: str(f))
def test_rows_up_to_sixteen(fa, fb, K):
    from paper_2310_10537_amd import binding as mx
    N = 72                                                # a last work-group of 8 columns
    g = torch.Generator(device="cuda").manual_seed(K + 8 * fa + fb)
    a = torch.randn((17, K), generator=g, device="cuda")
    b = torch.randn((N, K), generator=g, device="cuda")
    ea, sa = mx.mx_quantize(a, 1, fa)
    eb, sb = mx.mx_quantize(b, 1, fb)
    whole = mx.mx_gemm(ea, sa, fa, eb, sb, fb, K)
    for M in (1, 7, 8, 9, 15, 16):
        qa = mx.mx_quantize(a[:M].contiguous(), 1, fa)    # an operand of its own: rows beyond M are not there to be read
        for dt in (torch.float32, torch.bfloat16):
            got = mx.mx_gemm(qa[0], qa[1], fa, eb, sb, fb, K, dtype=dt)
            assert torch.equal(got.view(torch.uint8), whole[:M].to(dt).contiguous().view(torch.uint8)), (M, dt)
