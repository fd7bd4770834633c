"""The kernels that calls at the borders of the dispatch rules take, and the scratch memory they ask for (no GPU)."""
import pytest

import launches

P = 0x1000                                    # any aligned address
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def trace(tmp_path_factory):
    so = launches.build(str(tmp_path_factory.mktemp("runtime")))
    return lambda calls, refuse=0: launches.trace(so, [(n, a, refuse) for n, a in calls])


def names(seen):
    return [k[0] for k in seen]


def quantize(rows, cols, ld, dt, axis=1, fmt=0, rnd=0):
    return "mx_quantize", (P, dt, rows, cols, ld, axis, fmt, rnd, P, P, 0)


def test_long_dense_rows_are_one_run(trace):
    """Rows of which a 31-bit count of 16-byte pieces holds only a few: dense ones are one run whatever their length."""
    for dt, kernel in ((BF16, "cast_row_bf16_kernel"), (F32, "cast_row_f32_kernel")):
        for rows, cols in ((20, 1 << 30), (1, 1 << 35), (3, 1 << 33), (64, 4096)):
            (status, seen), = trace([quantize(rows, cols, cols, dt)])
            assert status == 0 and names(seen) == [kernel] and "true" in seen[0][1], (dt, rows, cols)
        # padded rows: a few launches of the same kernel
        (status, seen), = trace([quantize(20, 1 << 30, (1 << 30) + 8, dt)])
        assert status == 0 and 2 <= len(seen) <= 3 and set(names(seen)) == {kernel}, dt


def gemm(M, N, K, fa=0, fb=0, dt=F32):
    return "mx_gemm", (M, N, K, P, P, fa, P, P, fb, P, dt, N, 0)


def kernel_of(trace, *args, **kw):
    (status, seen), = trace([gemm(*args, **kw)])
    assert status == 0
    return names(seen)


def test_gemm_beyond_the_sizes_of_the_small_tiles(trace):
    long_k = (1 << 23) + 128
    staged, plain = "gemm_skinny_lds_kernel", "gemm_skinny_kernel"
    assert kernel_of(trace, 1, 64, long_k) == kernel_of(trace, 128, 64, long_k) == kernel_of(trace, 300, 64, long_k) == [staged]
    assert kernel_of(trace, 16, 64, (1 << 25) + 128) == kernel_of(trace, 300, 64, 1 << 26) == [plain]     # 32-bit offsets end
    assert kernel_of(trace, 100, 64, (1 << 23) + 32) == [plain]
    assert kernel_of(trace, 300, 64, (1 << 23) + 32) == ["gemm_direct_kernel"]
    # more than 2^36 entries of C: 256 x 256 tiles as far as those go, in 2^24 of them
    assert all("tile" in k for k in kernel_of(trace, 1 << 19, 1 << 19, 1024, dt=BF16))
    assert kernel_of(trace, (1 << 20) + 256, 1 << 20, 1024) == [staged]


def test_gemm_of_short_k(trace):
    direct, mid = ["gemm_direct_kernel"], ["gemm_mid_kernel"]
    E4M3, E3M2, E2M1 = 0, 2, 4
    for K in (32, 96, 224):
        assert kernel_of(trace, 593, 7040, K) == kernel_of(trace, 8192, 8192, K, E3M2, E2M1) == direct, K
    assert kernel_of(trace, 4096, 4096, 128) == kernel_of(trace, 8192, 8192, 128, E4M3, E2M1) == direct
    assert kernel_of(trace, 8192, 8192, 128) == mid                               # 8-bit pairs, many tiles
    assert kernel_of(trace, 593, 7040, 384, E3M2, E2M1) == direct and kernel_of(trace, 4096, 1536, 384, E3M2, E2M1) == mid
    assert kernel_of(trace, 1000, 1000, 256, E4M3, E2M1) == direct and kernel_of(trace, 593, 7040, 256, E4M3, E2M1) == mid
    assert kernel_of(trace, 1000, 1000, 256) == kernel_of(trace, 593, 1000, 512, E2M1, E2M1) == mid
    assert kernel_of(trace, 768, 2560, 288) == direct and kernel_of(trace, 768, 2560, 352) == mid
    assert kernel_of(trace, 593, 7040, 288, E4M3, E2M1) == direct and kernel_of(trace, 593, 7040, 416, E4M3, E2M1) == mid
    assert kernel_of(trace, 1 << 23, 64, 64) == mid                               # more rows than the direct grid holds


def gemm_qa(M, N, K, fa=0, fb=0, rnd=0):
    return "mx_gemm_qa", (M, N, K, P, K, fa, rnd, P, P, fb, P, BF16, N, 0)


def test_cast_on_load_of_short_k_in_registers(trace):
    kernel = "gemm_direct_qa_kernel"
    for M, N, K in ((300, 500, 160), (768, 2560, 256), (1000, 4096, 128), (129, 64, 288)):
        (status, seen), = trace([gemm_qa(M, N, K)])
        assert status == 0 and names(seen) == [kernel], (M, N, K)
    for M, N, K in ((300, 500, 512), (1000, 4096, 160), (4096, 1536, 256), (300, 500, 544), (128, 500, 96)):
        (status, seen), = trace([gemm_qa(M, N, K)])
        assert status == 0 and names(seen)[0] == "alloc" and kernel not in names(seen), (M, N, K)
    # scratch memory of the caller costs nothing: the line lies lower
    ws = 1 << 30
    for K, registers in ((64, True), (160, False)):
        call = "mx_gemm_qa_ws", (300, 500, K, P, K, 0, 0, P, P, 0, P, BF16, 500, P, ws, 0)
        (status, seen), = trace([call])
        assert status == 0 and "alloc" not in names(seen) and (kernel in names(seen)) == registers, K


def test_cast_on_load_when_scratch_is_refused(trace):
    """What never needed scratch memory does not fail without it; what always did still says so."""
    for M, N, K in ((300, 500, 4128), (1000, 4096, 160), (129, 64, 32), (5000, 64, 480)):
        for rnd in (0, 1):
            (status, seen), = trace([gemm_qa(M, N, K, rnd=rnd)], refuse=1)
            assert status == 0 and names(seen) == ["gemm_direct_qa_kernel"], (M, N, K)
    for call in (gemm_qa(300, 500, 4096), gemm_qa(128, 500, 4128), gemm_qa(300, 500, 4128, rnd=2), gemm_qa(300, 500, 4128, 5, 5)):
        (status, seen), = trace([call], refuse=1)
        assert status == 8 and seen == [], call
    (status, seen), = trace([gemm_qa(16, 500, 4096)], refuse=1)
    assert status == 0 and names(seen) == ["gemm_skinny_lds_kernel"]


def test_shapes_of_the_tile_tests_reach_their_kernels(trace):
    """tests/test_gpu_gemm_tiles.py on half-width and whole tiles, on an interior with a fringe, and cast on load by the tiles."""
    pytest.importorskip("torch")
    import test_gpu_gemm_tiles as t
    wide = ("gemm_tile_kernel", "gemm_tile16_kernel", "gemm_tile8_kernel")
    cases = [(shapes, half, shape, fa, fb) for shapes, half in ((t.HALF, True), (t.WHOLE, False), (t.INTERIOR, False))
             for shape in shapes for fa in range(5) for fb in range(5)]
    for (shapes, half, shape, fa, fb), (status, seen) in zip(cases, trace([gemm(*shape, fa, fb) for _, _, shape, fa, fb in cases])):
        name, args = seen[0][:2]
        assert status == 0 and name in wide, (shape, fa, fb)
        assert (name == "gemm_tile8_kernel" and args[-1] == "4") == half, (shape, fa, fb)           # four waves: half-width tiles
        assert len(seen) == (1 if shapes is not t.INTERIOR else 1 + (shape[0] % 256 > 0) + (shape[1] % 256 > 0)), shape
    M, N, K = t.NARROW
    (status, seen), = trace([gemm_qa(M, N, K)])
    assert status == 0 and seen[0][0] == "gemm_tile_kernel" and seen[0][1][3] == "true"       # casts on load
    assert names(seen)[1:] == ["alloc", "cast_row_bf16_kernel", "gemm_skinny_lds_kernel"]     # the last 32 rows


def test_interior_of_129_to_192_tiles(trace):
    E4M3, E3M2, E2M1 = 0, 2, 4
    one, two = (3100, 3072), (3340, 3340)                                          # 144 and 169 whole tiles
    for (M, N), K, fa, fb, interior in ((one, 4096, E4M3, E4M3, True), (one, 2048, E4M3, E4M3, False), (one, 1024, E3M2, E3M2, True),
                                        (one, 2048, E3M2, E2M1, True), (one, 4096, E4M3, E2M1, False), ((3100, 4096), 4096, E4M3, E2M1, True),
                                        (two, 4096, E4M3, E4M3, False), (two, 8192, E4M3, E4M3, True), (two, 4096, E3M2, E2M1, True),
                                        (two, 2048, E3M2, E3M2, False), (two, 8192, E2M1, E4M3, False), ((2600, 2560), 8192, E2M1, E2M1, False),
                                        ((2600, 2560), 4096, E3M2, E3M2, True), ((1568, 3584), 8192, E3M2, E3M2, True),
                                        ((1568, 3584), 8192, E2M1, E2M1, False), ((1568, 3584), 16384, E2M1, E2M1, True),
                                        ((1568, 3584), 16384, E4M3, E4M3, False)):
        (status, seen), = trace([gemm(M, N, K, fa, fb)])
        assert status == 0 and (seen[0][0] != "gemm_mid_kernel") == interior, (M, N, K, fa, fb)


def test_casts_of_few_rows_along_axis_0(trace):
    simple, away = "cast_col_simple_kernel", 1
    for rows, cols, dt, fmt, rnd, few in ((6, 400, F32, 0, 0, True), (24, 65536, F32, 4, 0, True), (24, 30000, F32, 4, 0, False),
                                          (32, 262144, F32, 2, away, True), (32, 65536, F32, 2, 0, False), (33, 262144, F32, 2, 0, False),
                                          (4, 1 << 21, BF16, 0, 0, False), (4, 1 << 21, BF16, 0, away, False), (4, 1 << 21, BF16, 5, 0, True),
                                          (16, 131072, BF16, 5, away, True), (12, 87376, BF16, 5, away, False), (12, 1 << 19, BF16, 5, 0, False),
                                          (6, 1 << 19, BF16, 3, away, True), (6, 1 << 19, BF16, 3, 0, False), (8, 1 << 17, BF16, 2, away, False), (8, 1 << 19, BF16, 4, away, True),
                                          (4, 248, F32, 0, 0, False)):
        (status, seen), = trace([quantize(rows, cols, cols, dt, 0, fmt, rnd)])
        assert status == 0 and len(seen) == 1 and (seen[0][0] == simple) == few, (rows, cols, dt, fmt, rnd)
    for rows, cols, few in ((10, 4096, True), (12, 65536, False), (12, 87384, True), (32, 32768, True), (33, 32768, False)):
        (status, seen), = trace([("mx_quantize_sr", (P, BF16, rows, cols, cols, 0, 0, 7, P, P, 0))])
        assert status == 0 and len(seen) == 1 and (seen[0][0] == simple) == few, (rows, cols)
