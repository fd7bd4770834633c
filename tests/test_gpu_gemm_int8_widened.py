"""MXINT8 products on the bf16 values of their blocks (whole tiles, and other sizes that the integer kernels take long for): routes and
scratch memory, ragged sizes, partial K steps, scale bytes at the ends of what bf16 and Float32 hold, the error of the sums."""
import pytest

import launches

INT8 = 5


def test_routes(tmp_path):
    rt = launches.build(str(tmp_path))
    P = 1 << 20

    def kernels(M, N, K, ws=True, refuse=0):
        call = ("mx_gemm_ws", (M, N, K, P, P, INT8, P, P, INT8, P, 1, N, P, 1 << 40, 0)) if ws else \
            ("mx_gemm", (M, N, K, P, P, INT8, P, P, INT8, P, 1, N, 0))
        (status, seen), = launches.trace(rt, [call + (refuse,)])
        return status, [k[0] + "".join(k[1][2:4]) if k[0] == "gemm_mid_kernel" else k[0] for k in seen]
    widen, large, short, check = "int8_widen_kernel", "gemm_mid_kernel22", "gemm_mid_kernel21", "gemm_int8_repair_kernel"
    staged, direct = "gemm_int8_lds_kernel", "gemm_int8_kernel"
    half = "gemm_bf16_half_kernel"
    # whole 256 x 256 tiles: 256 x 128 tiles where K is long, for whole rounds of them, and 128 x 128 tiles; other sizes: 128 x 64 tiles
    for M, N, K in ((8192, 4096, 4096), (2048, 3072, 2048), (4096, 4096, 2112), (5632, 4096, 2048)):
        assert kernels(M, N, K) == (0, [widen, half, check])
    for M, N, K in ((4096, 2304, 4096), (4096, 4608, 2112)):
        assert kernels(M, N, K) == (0, [widen, half, large, check])
    for M, N, K in ((4096, 4352, 512), (2048, 2048, 160), (4096, 4096, 1024), (4096, 4096, 2080)):
        assert kernels(M, N, K) == (0, [widen, large, check])
    for M, N, K in ((1000, 4096, 4096), (4100, 4352, 512), (8000, 6000, 416), (2048, 2048, 4096), (2847, 2624, 1248)):
        assert kernels(M, N, K) == (0, [widen, short, check])
    # ... where the kernels without scratch memory take long: five rounds and six of the staged one at K = 4096, scratch beyond 64 MB
    for M, N, K in ((128, 11008, 4096), (256, 4096, 4096), (1000, 1000, 4096), (748, 2432, 1408), (2048, 2048, 2048), (576, 4096, 4096), (6690, 801, 7168)):
        assert kernels(M, N, K) == (0, [staged])
    for M, N, K in ((256, 11008, 512), (300, 300, 96), (2847, 2112, 1248), (4806, 1099, 896), (1744, 9463, 512), (5251, 4911, 96), (8192, 8191, 224)):
        assert kernels(M, N, K) == (0, [direct])
    assert kernels(768, 3392, 4096) == (0, [staged]) and kernels(768, 3424, 4096) == (0, [widen, short, check])
    for M, N, K in ((8192, 4096, 4096), (1000, 4096, 4096)):                                    # by shape, wherever the scratch comes from
        assert kernels(M, N, K, ws=False)[1][1:] == kernels(M, N, K)[1]
    # refused scratch memory: an error where it always was one, the kernels without it elsewhere
    assert kernels(8192, 4096, 4096, ws=False, refuse=1)[0] != 0
    assert kernels(8000, 4000, 4096, ws=False, refuse=1) == (0, [staged])
    # K beyond 2^21 has never taken any
    assert kernels(2048, 2048, (1 << 21) + 32, ws=False, refuse=1) == (0, [direct])


def test_scratch_is_what_the_library_says(tmp_path):
    """The one allocation of a call is the bound that mx_gemm_workspace_bytes gives, and there is none where it gives 0."""
    from paper_2310_10537_amd import binding
    rt = launches.build(str(tmp_path))
    P = 1 << 20
    shapes = [(8192, 4096, 4096), (1000, 4096, 4096), (1001, 4099, 2080), (2304, 2816, 160), (300, 300, 96), (748, 2432, 1408), (128, 28672, 8192)]
    calls = [("mx_gemm", (M, N, K, P, P, INT8, P, P, INT8, P, 1, N, 0), 0) for M, N, K in shapes]
    for (M, N, K), (status, seen) in zip(shapes, launches.trace(rt, calls)):
        need = binding.mx_workspace_bytes("gemm", M, N, K, INT8, INT8)
        taken = [k[1] for k in seen if k[0] == "alloc"]
        assert status == 0 and taken == ([need] if need else []), (M, N, K)


def test_scratch_of_the_binding(monkeypatch):
    """From torch's allocator on the current stream, outside a capture, for the sizes whose route uses it."""
    import types

    import torch
    from paper_2310_10537_amd import binding
    cpu, capturing = torch.device("cpu"), [False]
    current = types.SimpleNamespace(device=cpu, cuda_stream=11)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: current)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing[0])
    monkeypatch.setattr(torch, "empty", lambda n, dtype, device: n)                            # (gigabytes otherwise)

    def size(M, N, K, stream=None, kind="gemm"):
        return binding._int8_workspace(kind, M, N, K, cpu, stream)
    assert size(8192, 4096, 4096) == binding.mx_workspace_bytes("gemm", 8192, 4096, 4096, INT8, INT8)
    assert size(1000, 4096, 4096, kind="gemm_q") == binding.mx_workspace_bytes("gemm_q", 1000, 4096, 4096, INT8, INT8)
    assert size(4100, 4352, 512) is not None and size(2048, 2048, 512) is not None
    for shape in ((128, 28672, 8192), (256, 4096, 4096), (300, 300, 96), (2100, 2100, 512)):     # (64 tiles in the last, not whole ones)
        assert size(*shape) is None
    assert binding._qa_workspace(1000, 4096, 4096, INT8, INT8, cpu, None) == binding.mx_workspace_bytes("gemm_qa", 1000, 4096, 4096, INT8, INT8)
    assert size(8192, 4096, 4096, types.SimpleNamespace(cuda_stream=12)) is None
    capturing[0] = True
    assert size(8192, 4096, 4096) is None


# 128 x 64 tiles, 128 x 128, 256 x 128 with and without others beside them; K with a partial step
SHAPES = [(330, 12320, 2048), (1000, 4610, 2048), (520, 4103, 4640), (4100, 4360, 544), (4096, 4352, 576), (2304, 3840, 160),
          (4096, 2304, 2112), (2048, 4096, 2240)]
SUMS = [(4096, 4096, 4096), (2048, 2304, 512), (2048, 2048, 160), (1000, 4096, 4096), (2000, 4100, 1024), (700, 2600, 8192),
        (8192, 2200, 512), (3000, 2000, 2080)]
TWO = [(1000, 4610, 2048), (4096, 4096, 512), (2048, 4096, 2048)]


def test_shapes_below_take_the_values():
    from paper_2310_10537_amd import binding
    for M, N, K in SHAPES + SUMS + TWO:
        assert binding.mx_workspace_bytes("gemm", M, N, K, INT8, INT8) > 0, (M, N, K)


def operand(torch, g, rows, K, lo, hi):
    q = torch.randint(-128, 128, (rows, K), generator=g, device="cuda", dtype=torch.int32)
    s = torch.randint(lo, hi + 1, (rows, K // 32), generator=g, device="cuda", dtype=torch.int32)
    q[0, :32], s[0, 0] = 0, 0                                     # zeros: their scale does not count
    q[1, 32:64], s[1, 1] = -128, hi
    q[2, :] = 127
    return q.to(torch.int8), s.to(torch.uint8)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("ranges", [((120, 134), (120, 134)), ((7, 20), (133, 160)), ((180, 253), (60, 125)),            # held by bf16
                                    ((6, 20), (133, 160)), ((60, 79), (60, 79)), ((200, 254), (60, 120)), ((180, 200), (180, 200)),
                                    ((0, 12), (120, 160))])
def test_against_float64(shape, ranges):
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    (qa, sa), (qb, sb) = operand(torch, g, M, K, *ranges[0]), operand(torch, g, N, K, *ranges[1])
    C = mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K)
    rows = torch.cat([torch.arange(3), torch.randint(0, M, (29,), generator=torch.Generator().manual_seed(1)), torch.tensor([M - 1])]).cuda()

    def value(q, s):
        return q.double() * torch.exp2(s.double() - 133).repeat_interleave(32, dim=1)
    a, b = value(qa[rows], sa[rows]), value(qb, sb)
    ref, mag = a @ b.T, a.abs() @ b.abs().T
    got = C[rows].double()
    big = torch.finfo(torch.float32).max
    inside = mag < big / 4                                        # beyond: a sum of Float32 numbers overflows on the way, or not
    # every block sum is exact or a few roundings of 2^-24 of the running sum, K / 16 steps of the instruction at most; below, the
    # spacing of Float32's denormal numbers once per block
    tol = mag * (K / 16 * 2.0 ** -24) + K / 32 * 2.0 ** -149
    assert bool(((got - ref).abs() <= tol)[inside].all()), float(((got - ref).abs() / mag.clamp_min(1e-300))[inside].max())
    assert bool((~torch.isfinite(got) | (got.abs() > big / 1e6))[ref.abs() > big * 2].all())


# n Float32 additions of terms of random sign, one behind the other, leave a relative error of 2.4e-8 (n / 2)^0.5 in the 2-norm (a sum of k
# terms is of the order of k^0.5, a rounding errs by 2^-24 times 0.41 in the mean square).  The integer kernels add a wave's K / 256 block sums
# and then eight waves' sums, or (short K, or no multiple of 128) K / 32 block sums; the chains of E2M3 halves that whole tiles had, K / 16 terms.
@pytest.mark.gpu
@pytest.mark.parametrize("shape", SUMS, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("signs", ["random", "one"])
def test_sums_err_no_more_than_block_sums_do(shape, signs):
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(M + 3 * N + K)

    def operand(rows):                                            # scales over 16 octaves: sums that Float32 rounds
        x = torch.randn((rows, K), generator=g, device="cuda")
        x = x * torch.exp2(torch.randint(-8, 8, (rows, K // 32), generator=g, device="cuda").float()).repeat_interleave(32, dim=1)
        return mx.mx_quantize((x.abs() if signs == "one" else x).to(torch.bfloat16), 1, INT8)
    (qa, sa), (qb, sb) = operand(M), operand(N)
    C = mx.mx_gemm(qa, sa, INT8, qb, sb, INT8, K)

    def value(q, s):
        return q.view(torch.int8).double() * torch.exp2(s.double() - 133).repeat_interleave(32, dim=1)
    ref = value(qa[:256], sa[:256]) @ value(qb, sb).T
    err = float((C[:256].double() - ref).norm() / ref.norm())
    whole = M % 256 == 0 and N % 256 == 0 and (M // 256) * (N // 256) >= 64
    terms = K / 16 if whole else K / 32 if K % 128 or K < 1024 else K / 256 + 8
    # with one sign the sums grow evenly: (n / 3)^0.5 roundings of the whole, less than above
    assert err <= 1.1 * 2.4e-8 * (terms / 2) ** 0.5, err


@pytest.mark.gpu
@pytest.mark.parametrize("zeros", [False, True])
def test_nan_scales(zeros):
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = 1000, 4610, 2048
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    (qa, sa), (qb, sb) = operand(torch, g, M, K, 120, 130), operand(torch, g, N, K, 120, 130)
    sa[700, 3] = 255
    sb[2049, 31] = 255
    if zeros:
        qa[700, 96:128] = 0
        qb[2049, 992:1024] = 0
    C = mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K)
    nan = torch.isnan(C)
    assert bool(nan[700].all()) and bool(nan[:, 2049].all()) and int(nan.sum()) == M + N - 1


def spread(torch, g, rows, K, lo=120, hi=136):
    q = torch.randint(-127, 128, (rows, K), generator=g, device="cuda", dtype=torch.int32).to(torch.int8)
    return q, torch.randint(lo, hi, (rows, K // 32), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", TWO, ids=lambda s: "x".join(map(str, s)))
def test_a_block_out_of_the_ordinary_leaves_the_other_rows_alone(shape):
    """A NaN scale, scales near 0, at the largest value of a block and at the end of Float32's range: the entries of rows and columns in
    other 64 x 64 tiles keep their bits."""
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(K)
    (qa, sa), (qb, sb) = spread(torch, g, M, K), spread(torch, g, N, K)

    def product():
        return mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K)

    def value(q, s):
        return q.double() * torch.exp2(s.double() - 133).repeat_interleave(32, dim=-1)
    plain, c = product(), slice(3900, 4096)
    for scale, q in ((255, 1), (0, 3), (3, -128), (6, 127), (253, 1), (254, -128)):
        sa[130, 5], qa[130, 160:192] = scale, q
        sb[4000, 5] = 60                                          # (with the largest ones a product below 2^127)
        got = product()
        keep = torch.ones((M, N), dtype=torch.bool, device="cuda")
        keep[130], keep[:, 4000] = False, False
        if scale in (253, 254):                                   # recomputed: the tiles of rows 128 .. 191
            keep[128:192] = False
        assert torch.equal(got[keep], plain[keep]), scale
        if scale == 255:
            assert bool(torch.isnan(got[130]).all()) and int(torch.isnan(got).sum()) == N
            continue
        x, y = value(qa[130], sa[130]), value(qb[c], sb[c])
        ref, mag = y @ x, y.abs() @ x.abs()
        inside = ref.abs() < 2.0 ** 127
        assert bool(((got[130, c].double() - ref).abs() <= mag * K * 2.0 ** -24)[inside].all()), scale
        assert bool((torch.isinf(got[130, c]) | (got[130, c].abs() > 2.0 ** 126))[~inside].all()), scale
        assert scale < 253 or bool(inside[100])


@pytest.mark.gpu
@pytest.mark.parametrize("shape,total", [(TWO[0], 366), (TWO[0], 378), (TWO[0], 379), (TWO[1], 378), (TWO[1], 379), (TWO[2], 378)], ids=str)
def test_sums_that_cancel_inside_a_block(shape, total):
    """Sixteen products of 2^14 times the scales of one sign, then sixteen of the other: the block's sum is zero, and so it stays
    where the sum of half of them is beyond Float32 (or, in sums of one block at a time, so large that it would wipe out the others)."""
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(total)
    (qa, sa), (qb, sb) = spread(torch, g, M, K), spread(torch, g, N, K)

    def product():
        return mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K)[200:232, 300:340]
    qa[200:232, 64:96], qb[300:340, 64:96] = 0, 0
    without = product()
    qa[200:232, 64:80], qa[200:232, 80:96], qb[300:340, 64:96] = 127, -127, 127
    sa[200:232, 2], sb[300:340, 2] = total - 185, 185
    got = product()
    tol = float(without.square().mean().sqrt()) * 100 * K * 2.0 ** -24       # (the other blocks' sums in another order of magnitude at most)
    assert bool(torch.isfinite(got).all()) and float((got - without).abs().max()) <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(4096, 2304, 2112), (2048, 4096, 2240), (2048, 3072, 2048), (4096, 4096, 576), (1000, 4610, 2080)], ids=str)
@pytest.mark.parametrize("dt", ["float32", "bfloat16"])
def test_exact_integers_in_rows_of_any_pitch(shape, dt):
    """Every sum is a whole number that Float32 holds, whatever the order: entries that differ are in the wrong place."""
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    dt = getattr(torch, dt)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    qa, qb = (torch.randint(-50, 51, (r, K), generator=g, device="cuda", dtype=torch.int32).to(torch.int8) for r in (M, N))
    sa, sb = (torch.full((r, K // 32), 130, dtype=torch.uint8, device="cuda") for r in (M, N))       # 2^3 / 64 each
    want = (qa.float() @ qb.float().T / 64).to(dt)                # (whole numbers below 2^24 as well)
    assert K * 2500 < 1 << 24
    for pitch in (N, N + 3, N + 8):
        buf = torch.full((M, pitch), 7.0, dtype=dt, device="cuda")
        mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K, out=buf[:, :N])
        assert torch.equal(buf[:, :N], want) and bool((buf[:, N:] == 7.0).all()), pitch


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1000, 4096, 4096), (2048, 4096, 2048)], ids=str)
def test_captured(shape):
    """A capture takes the scratch memory into the graph: every replay gives the eager bits, with eager products and new tensors between."""
    import torch
    from paper_2310_10537_amd import binding as mx
    M, N, K = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    (qa, sa), (qb, sb) = spread(torch, g, M, K), spread(torch, g, N, K)
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")

    def product(out=None):
        return mx.mx_gemm(qa.view(torch.uint8), sa, INT8, qb.view(torch.uint8), sb, INT8, K, dtype=torch.bfloat16, out=out)
    product(out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        product(out)
    need = mx.mx_workspace_bytes("gemm", M, N, K, INT8, INT8)
    later = [torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(3)]
    for seed in range(4):
        qa.copy_(torch.roll(qa, 1, 0))                            # the graph reads what the operands hold now
        want = product()
        out.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and all(bool((t == 0xA5).all()) for t in later), seed
