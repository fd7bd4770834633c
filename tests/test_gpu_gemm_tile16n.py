"""The 256 x 256 tiles of 6- / 4-bit pairs on the 16 x 16 x 128 instruction against the small-tile kernel (which the instruction model
holds to its bits): every pair, one to many trips of four K steps, row pitches with and without wide stores.  The problems
around them -- K no multiple of 512, fewer tiles, 4-bit pairs -- stay with the other kernels (checked without a GPU)."""
import pytest

import launches

PAIRS = [(2, 2), (2, 3), (3, 2), (3, 3), (2, 4), (3, 4), (4, 2), (4, 3)]
SHAPES = [(4096, 3584, 6144), (3584, 4352, 6656)]              # 224 tiles and twelve trips; 238 tiles and thirteen


def test_route(tmp_path):
    rt = launches.build(str(tmp_path))
    P = 1 << 20

    def kernel(M, N, K, fa, fb):
        (status, seen), = launches.trace(rt, [("mx_gemm", (M, N, K, P, P, fa, P, P, fb, P, 1, N, 0), 0)])
        assert status == 0
        return seen[0][0]
    for fa, fb in PAIRS:
        for M, N, K in SHAPES:
            assert kernel(M, N, K, fa, fb) == "gemm_tile16_kernel", (fa, fb, M, N, K)
        assert kernel(4096, 3584, 6144 + 128, fa, fb) == "gemm_tile8_kernel"
        assert kernel(4096, 3328, 8192, fa, fb) == "gemm_tile8_kernel"                    # 208 tiles
        assert kernel(4096, 3584, 4096, fa, fb) == ("gemm_tile16_kernel" if 4 not in (fa, fb) else "gemm_tile8_kernel")
        assert kernel(4096, 3584, 3584, fa, fb) == "gemm_tile8_kernel"
    assert kernel(4096, 4096, 8192, 4, 4) == "gemm_tile8_kernel"


@pytest.mark.gpu
@pytest.mark.parametrize("fa,fb", PAIRS, ids=lambda v: str(v))
def test_same_bits_as_small_tiles(fa, fb):
    import torch
    from paper_2310_10537_amd import binding as mx
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * fa + fb)
    for n, (M, N, K) in enumerate(SHAPES):
        def operand(rows, fmt):
            x = torch.randn((rows, K), generator=g, device="cuda")
            x = x * torch.exp2(torch.randint(-6, 6, (rows, K // 32), generator=g, device="cuda").float()).repeat_interleave(32, dim=1)
            return mx.mx_quantize(x.to(torch.bfloat16), 1, fmt)
        (ae, as_), (be, bs) = operand(M, fa), operand(N, fb)
        dt = (torch.float32, torch.bfloat16)[(n + fa + fb) % 2]
        C = mx.mx_gemm(ae, as_, fa, be, bs, fb, K, dtype=dt)
        rows, cols = torch.arange(0, M, 512), torch.arange(0, N, 512)
        for r, c in [(int(rows[k % len(rows)]), int(cols[(3 * k + 1) % len(cols)])) for k in range(8)]:
            h, w = min(512, M - r), min(512, N - c)                     # at most 64 tiles of 64 x 64: the small-tile kernel
            part = mx.mx_gemm(ae[r:r + h], as_[r:r + h], fa, be[c:c + w], bs[c:c + w], fb, K, dtype=dt)
            assert torch.equal(C[r:r + h, c:c + w], part), (M, N, K, r, c)
        pad = 2 if dt == torch.float32 else 6                          # a row pitch that rules out the wide stores
        buf = torch.full((M, N + pad), 7.0, dtype=dt, device="cuda")
        mx.mx_gemm(ae, as_, fa, be, bs, fb, K, out=buf[:, :N])
        assert torch.equal(buf[:, :N], C) and bool((buf[:, N:] == 7.0).all())
