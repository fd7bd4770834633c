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
