"""The 256 x 256 tiles of 6- / 4-bit pairs on the 16 x 16 x 128 instruction against the small-tile kernel (which the instruction model
holds to its bits): every pair, the fewest trips of four K steps and more, even and odd, row pitches with and without wide stores, scale bytes
from one end to the other.  The problems around them -- K no multiple of 512, fewer tiles, a last round of tiles that leaves much of the
chip idle, 4-bit pairs -- stay with the other kernels (checked without a GPU)."""
import pytest

import launches

PAIRS = [(2, 2), (2, 3), (3, 2), (3, 3), (2, 4), (3, 4), (4, 2), (4, 3)]
SHAPES = [(4096, 4096, 6144), (3840, 4096, 8704)]              # 256 tiles and twelve trips; 240 tiles and seventeen


def test_route(tmp_path):
    rt = launches.build(str(tmp_path))
    P = 1 << 20

    def kernel(tiles_m, tiles_n, K, fa, fb):
        (status, seen), = launches.trace(rt, [("mx_gemm", (256 * tiles_m, 256 * tiles_n, K, P, P, fa, P, P, fb, P, 1, 256 * tiles_n, 0), 0)])
        assert status == 0 and seen[0][3] == (256 if seen[0][0] == "gemm_tile16_kernel" else 512)     # four waves or eight
        assert seen[0][1][:2] == (str(fa), str(fb))
        return seen[0][0] == "gemm_tile16_kernel"
    for fa, fb in PAIRS:
        for M, N, K in SHAPES:
            assert kernel(M // 256, N // 256, K, fa, fb), (fa, fb, M, N, K)
        assert not kernel(16, 16, 6144 + 128, fa, fb)
        assert not kernel(16, 13, 12288, fa, fb)                                          # 208 tiles
        assert not kernel(16, 16, 3584, fa, fb)
        # the last round of tiles: full, 176 of 256 behind one full round or four or seven, 240
        line = [[kernel(*tiles, K, fa, fb) for K in (4096, 6144, 8192)] for tiles in ((16, 32), (16, 27), (30, 40), (44, 45), (31, 16))]
        if fa != 4 and fb != 4:
            assert line == [[True] * 3, [False, True, True], [True] * 3, [True] * 3, [True] * 3]
        elif fa == 4:
            assert line == [[False, True, True], [False, False, True]] + [[False, True, True]] * 3
        else:
            assert line == [[False, True, True], [False] * 3, [False] * 3, [False, False, True], [False, True, True]]
    assert not kernel(16, 16, 8192, 4, 4)


@pytest.mark.gpu
@pytest.mark.parametrize("fa,fb", PAIRS, ids=lambda v: str(v))
def test_same_bits_as_small_tiles(fa, fb):
    import torch
    from paper_2310_10537_amd import binding as mx
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * fa + fb)
    six = [(4096, 4096, 4096), (3840, 4096, 4608)] if 4 not in (fa, fb) else []          # eight and nine trips
    for n, (M, N, K) in enumerate(SHAPES + six):
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


@pytest.mark.gpu
@pytest.mark.parametrize("fa,fb", PAIRS, ids=lambda v: str(v))
def test_same_bits_with_any_scale_bytes(fa, fb):
    """Scale bytes from 0 to 254 that differ from block to block, NaN scales, rows of zeros and of the largest codes."""
    import torch
    from paper_2310_10537_amd import binding as mx
    g = torch.Generator(device="cuda")
    g.manual_seed(100 * fa + fb)
    M, N, K = SHAPES[0]

    def operand(rows, fmt, centre):
        e = torch.randint(0, 256, (rows, K * mx.FORMAT_BITS[fmt] // 8), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)
        s = torch.randint(centre - 12, centre + 13, (rows, K // 32), generator=g, device="cuda", dtype=torch.int32)
        any_ = torch.randint(0, 255, (rows, K // 32), generator=g, device="cuda", dtype=torch.int32)
        kind = torch.arange(rows, device="cuda") % 37
        s[kind == 1], e[kind == 2], e[kind == 3] = any_[kind == 1], 0, 255
        s[kind == 4, 17], s[kind == 5, 80], s[kind == 6, K // 32 - 1] = 255, 254, 0
        return e, s.to(torch.uint8)
    for ca, cb in ((127, 127), (12, 120), (242, 130)):
        (ae, as_), (be, bs) = operand(M, fa, ca), operand(N, fb, cb)
        C = mx.mx_gemm(ae, as_, fa, be, bs, fb, K)
        assert bool(torch.isnan(C[4]).all()) and not bool(torch.isnan(C[0, :4]).any()) or ca == 242
        for r, c in ((0, 512), (1536, 0), (3584, 3584)):
            part = mx.mx_gemm(ae[r:r + 512], as_[r:r + 512], fa, be[c:c + 512], bs[c:c + 512], fb, K)
            assert torch.equal(C[r:r + 512, c:c + 512].view(torch.int32), part.view(torch.int32)), (ca, cb, r, c)
