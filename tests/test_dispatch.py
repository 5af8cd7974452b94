"""The dispatch rules at the sizes where they change, and over the launch
limits (no GPU needed)."""
import pytest

from tests.dispatch_util import (gather_cols, gather_cols_sparse, gather_rows_single, gemm_plan, gemv, launches,
                                 mask_route, unmask_words)

MAX_THREADS = 2 ** 32 - 256


@pytest.mark.parametrize("cols", [1, 3, 5, 17, 63, 127, 191])
def test_many_short_ragged_rows_take_the_general_kernel(cols):
    """One workgroup per row left 4 to 48 of 256 threads at work."""
    for rows in (65537, 2 ** 20):
        assert mask_route(rows, cols, x="rows") == "general"
        assert mask_route(rows, cols, noise="rows", digits=True) == "general"
    assert mask_route(512, cols, x="rows", noise="rows") == "ragged"


def test_ragged_and_aligned_rows():
    assert mask_route(2 ** 20, 192, x="rows", aligned=False) == "ragged"
    assert mask_route(6144, 16, x="rows") == "ragged" and mask_route(6145, 16, x="rows") == "general"
    assert mask_route(2048, 15, x="rows") == "ragged" and mask_route(2049, 15, x="rows") == "general"
    assert mask_route(2 ** 20, 4, x="rows", aligned=True) == "quad"
    assert mask_route(4096, 4096, x="strided") == "general"
    assert mask_route(4096, 4096, x="rows", noise="turned") == "general"


@pytest.mark.parametrize("aligned", [False, True])
@pytest.mark.parametrize("digits", [False, True])
def test_row_kernels_stay_within_a_launch(aligned, digits):
    """Calls of up to 2^32 threads of the general kernel are accepted; a kernel
    with a workgroup per row takes them only if its own grid fits too."""
    for cols in (3, 64, 192, 1025, 4096, 2 ** 20):
        lanes = 64 * -(-cols // 64) // 4 if digits else 4 * -(-cols // 16)
        per_row = 256 * -(-lanes // 256)
        fit = MAX_THREADS // per_row
        for rows in (fit, fit + 1, 20_000_000):
            r = mask_route(rows, cols, x="rows", aligned=aligned, digits=digits)
            if r in ("quad", "ragged"):
                assert rows * per_row <= MAX_THREADS
            assert rows > fit or cols < 192 or r == ("quad" if aligned else "ragged")


@pytest.mark.parametrize("rows,cols,x,noise", [
    (1, 2 ** 20, None, "turned"), (2, 2 ** 20, "turned", None), (2 ** 20, 3, "turned", None), (65, 512, None, "turned"),
    (8, 262144, "turned", "turned"), (1, 4096, None, "turned"), (33, 262144, None, "turned")])
def test_turned_matrices_with_a_short_side(rows, cols, x, noise):
    """64 x 64 tiles of which most is empty took up to 13 times as long."""
    assert mask_route(rows, cols, x=x, noise=noise, digits=True) == "general"


def test_turned_matrices():
    assert mask_route(4096, 1536, x="turned", noise="turned") == "turn"
    assert mask_route(1536, 4096, noise="turned", digits=True) == "turn"
    assert mask_route(64, 64, x="turned") == "turn" and mask_route(2, 6, x="turned") == "turn"
    assert mask_route(127, 2 ** 15, noise="turned") == "general" and mask_route(129, 2 ** 15, noise="turned") == "turn"
    assert mask_route(12, 2 ** 20, x="turned") == "turn" and mask_route(11, 2 ** 20, x="turned") == "general"
    assert mask_route(2 ** 20, 17, x="turned") == "turn" and mask_route(2 ** 20, 16, x="turned") == "general"
    assert mask_route(2 ** 40, 2 ** 30, x="turned") == "general"     # more tiles than a launch has workgroups
    assert mask_route(4096, 4096, x="turned", noise="rows") == "general"


def test_products_of_one_or_two_rows():
    """Dot products only where they are ahead: not on few long rows of B, many
    short ones, or a single chunk of columns."""
    for M, N, K in ((1, 1024, 5120), (1, 64, 4096), (1, 200, 6144), (1, 28672, 128), (2, 16384, 256), (3, 4096, 1536),
                    (1, 8192, 6208), (2, 4096, 2112)):
        assert not gemv(M, N, K, unmask=False)
    for M, N, K in ((1, 4096, 1536), (1, 1024, 4096), (1, 3072, 6144), (1, 64, 3072), (2, 8192, 2048), (1, 28672, 512),
                    (1, 8192, 64)):
        assert gemv(M, N, K, unmask=False)
    for M, N, K in ((1, 28672, 64), (2, 4096, 64), (1, 64, 6208), (2, 64, 2112), (3, 64, 128), (1, 2 ** 27 - 7, 128)):
        assert not gemv(M, N, K, unmask=True)
    for M, N, K in ((1, 64, 65), (1, 28672, 6144), (2, 16384, 2048)):
        assert gemv(M, N, K, unmask=True)
    for unmask in (False, True):        # a workgroup of 256 threads per 8 rows of B
        assert gemv(1, 2 ** 27 - 8, 512, unmask) and not gemv(1, 2 ** 27 - 7, 512, unmask)


def test_unmask_from_words():
    """Two waves per workgroup only while the inner dimension is short, or the
    workgroups are many for one tile each."""
    for M, N, K, want in ((16, 4096, 4096, (1, 4)), (3, 4097, 1024, (1, 2)), (8, 5003, 1025, (2, 4)), (9, 4097, 64, (2, 4)),
                          (8, 8192, 4096, (2, 4)), (8, 8193, 4096, (1, 2)), (8, 12288, 64, (1, 2)), (16, 12288, 704, (2, 4)),
                          (3, 12289, 64, (2, 4)), (16, 12289, 65, (2, 2)), (16, 28672, 3072, (2, 2)),
                          (3, 16384, 3073, (2, 4)), (8, 12288, 6145, (2, 4))):
        assert unmask_words(M, N, K) == want, (M, N, K)


def test_column_gathers():
    """Eight rows of d staged by a handful of workgroups, and wide or narrow
    matrices staged whole, had taken up to twice the single gather's time."""
    for M, N, want in ((16, 1024, 1), (17, 1024, 2), (1, 4096, 1), (5, 4096, 2), (8, 4096, 2), (16, 4096, 4), (8, 8192, 4),
                       (16, 8192, 8), (17, 8192, 8), (2, 8193, 2), (3, 8193, 4), (8, 14336, 8), (200, 256, 4)):
        assert gather_cols(1, M, N, 1536) == want and gather_cols(2, M, N, 1536) == want, (M, N)
    for nterms, M, N, cols, want in ((1, 8, 28672, 512, 0), (2, 8, 28672, 512, 8), (1, 8, 28672, 513, 8), (1, 8, 8192, 4096, 0),
                                     (1, 16, 8192, 4096, 4), (1, 64, 8192, 8192, 0), (1, 64, 14336, 8192, 2),
                                     (1, 200, 28672, 8193, 0), (1, 200, 28672, 2 ** 20, 0)):
        assert gather_cols(nterms, M, N, cols) == want, (M, N, cols)
    for M in (1, 2, 3, 7, 8, 64, 1000):
        for N in (1, 33, 8192, 8193, 10 ** 6):
            for cols in (1, 513, 2560, 2561, 5121, 8192, 20480, 20481):
                assert 4 * cols * gather_cols(2, M, N, cols) <= 80 * 1024


def test_column_gathers_of_few_entries():
    """Staging d's rows for a few entries per row took up to twice the single
    gather's time."""
    for n, M, N, cols, entries in ((1, 64, 8192, 1536, 4), (1, 1, 1024, 1536, 12), (1, 64, 14336, 1024, 16),
                                   (2, 64, 8192, 2560, 8)):
        assert gather_cols_sparse(n, M, N, cols, entries)
    for n, M, N, cols, entries in ((1, 64, 8192, 1536, 24), (1, 64, 14336, 1536, 20), (2, 64, 28672, 2560, 40),
                                   (2, 8, 8192, 2560, 8), (2, 16, 14336, 2560, 160), (1, 64, 8192, 4096, 4)):
        assert not gather_cols_sparse(n, M, N, cols, entries)


def test_row_gathers():
    """A single matrix of few outputs or few entries per row, and long launches
    over sparse rows, had become slower with all matrices at once."""
    for n, weight, entries, rows, ncols in ((1, 1, 80, 1, 8192), (1, 1, 80, 8, 5000), (1, 1, 16, 64, 8192), (1, 0, 4, 200, 32768),
                                            (1, 0, 24, 200, 8192), (1, 0, 24, 7, 8192), (2, 0, 48, 200, 18432),
                                            (1, 0, 256, 1, 8192)):
        assert gather_rows_single(n, weight, entries, rows, ncols)
    for n, weight, entries, rows, ncols in ((1, 1, 80, 16, 5000), (1, 1, 256, 1, 8192), (1, 0, 24, 8, 8192), (2, 0, 40, 8, 18432),
                                            (2, 1, 160, 200, 32768), (2, 1, 160, 1, 512), (1, 0, 256, 64, 8192)):
        assert not gather_rows_single(n, weight, entries, rows, ncols)


def test_tiled_products_where_64_row_tiles_were_behind():
    """A few tiles left over after whole turns of the units, and one and a bit
    turns of many stages: 3-13% slower than with 128-row tiles."""
    for M, N, K, epi in ((640, 6539, 4096, "store"), (640, 6539, 2560, "store"), (448, 14336, 2560, "store"),
                         (333, 11008, 2560, "store"), (384, 11008, 2560, "store"), (448, 9728, 8192, "store"),
                         (192, 14336, 8192, "store"), (160, 14336, 4096, "unmask"), (448, 6539, 8192, "store")):
        assert gemm_plan(M, N, K, epi)[0] == "128", (M, N, K, epi)


def test_tiled_products():
    for M, N, K, epi, want in ((200, 4608, 1536, "unmask", ("64k", 0, 1)), (200, 6144, 4096, "store", ("64k", 0, 1)),
                               (333, 14336, 1536, "unmask", ("64", 0, 1)), (1024, 6144, 1536, "store", ("64", 0, 1)),
                               (28672, 8192, 1536, "store", ("128", 0, 1)), (2048, 28672, 8192, "store", ("128", 0, 1)),
                               (128, 4608, 0, "store", ("64k", 0, 1))):
        assert gemm_plan(M, N, K, epi) == want, (M, N, K, epi)
    for M in (65, 200, 333, 2048):
        for N in (1, 5003, 28672):
            for K in (64, 704, 8192):
                assert gemm_plan(M, N, K, "unmask")[1:] == (0, 1)      # needs whole products
                for epi in ("store", "accum"):
                    form, tiles, k = gemm_plan(M, N, K, epi)
                    assert k == 1 or (form == "128" and 0 < 2 * tiles < 256 and K >= 128 * k)


@pytest.mark.parametrize("rows,units,most", [(5, 3, 100), (5, 3, 15), (5, 3, 14), (5, 3, 3), (5, 7, 3), (1, 1, 1), (4, 8, 7)])
def test_launches_cover_the_rows_once(rows, units, most):
    seen = set()
    for r, nr, u, nu in launches(rows, units, most):
        assert nr * nu <= most
        part = {(i, j) for i in range(r, r + nr) for j in range(u, u + nu)}
        assert len(part) == nr * nu and not part & seen
        seen |= part
    assert seen == {(i, j) for i in range(rows) for j in range(units)}


def test_launches_of_long_rotations():
    """2^22 blocks of 16384 on 1024 threads, 2^31 of 16 on four: past a launch."""
    for rows, units, threads in ((2 ** 22, 1, 1024), (1, 2 ** 22, 1024), (2 ** 22, 512, 4), (3, 2 ** 30, 4)):
        parts = launches(rows, units, MAX_THREADS // threads)
        assert len(parts) > 1 and sum(nr * nu for _, nr, _, nu in parts) == rows * units
        assert all(nr * nu * threads <= MAX_THREADS for _, nr, _, nu in parts)
    assert launches(2 ** 20, 2, MAX_THREADS // 1024) == [(0, 2 ** 20, 0, 2)]
    assert launches(10, 4, 4, stop_after=3)[-1] == (2, 1, 0, 4)
