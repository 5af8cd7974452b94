"""The gathers over several sparse matrices in one call, against the oracle's
products: SPARSE and WEIGHT levels side by side, the levels that are left to
the single gathers (long rows, wide matrices), empty levels, rows of d and
widths around the kernels' groups, unaligned rows."""
import numpy as np
import pytest
import torch

from oracle import sampling as smp
from oracle.ring import ring_add, ring_matmul, ring_sub
from tests.gpu_util import to_dev_ring, to_np_u32

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_29221_amd import mosaic as m

# (kind, columns, parameter): entries per row for weight, s of density 2^-s for sparse
LEVELS = {
    "weights": [("weight", 300, 80), ("weight", 128, 128)],
    "mixed": [("sparse", 700, 3), ("weight", 64, 9), ("sparse", 2048, 0)],
    "one": [("sparse", 65, 2)],
    "four": [("weight", 40, 40), ("sparse", 257, 1), ("weight", 1024, 80), ("sparse", 5, 31)],
    "empty": [("weight", 30, 0), ("sparse", 90, 4)],
    "long": [("weight", 600, 257), ("sparse", 3000, 4)],
    "wide": [("sparse", 17000, 7), ("weight", 50, 3)],
}


def _levels(name, rows):
    out = []
    for k, (kind, cols, p) in enumerate(LEVELS[name]):
        if kind == "weight":
            rr = m.rng(8, 0x60 + k, 3, m.DIST_WEIGHT, row_weight=p)
            P = smp.sample_matrix("weight", rows, cols, 8, 0x60 + k, 3, row_weight=p)
        else:
            rr = m.rng(8, 0x60 + k, 3, m.DIST_SPARSE, log2_inv_density=p)
            P = smp.sample_matrix("sparse", rows, cols, 8, 0x60 + k, 3, log2_inv_density=p)
        out.append((rr, cols, P))
    return out


@pytest.mark.parametrize("name", list(LEVELS))
@pytest.mark.parametrize("rows,ncols", [(1, 1), (3, 255), (2, 258), (9, 1000)])
def test_stream_gather_rows_terms(name, rows, ncols):
    rng = np.random.default_rng(rows * 17 + ncols)
    terms, want = [], rng.integers(0, 2 ** 32, (rows, ncols), dtype=np.uint32)
    c = torch.full((rows, ncols + 3), 7, dtype=torch.int32, device="cuda")
    c[:, 1: 1 + ncols] = to_dev_ring(want)
    subtract = bool(ncols % 2)
    for rr, cols, P in _levels(name, rows):
        D = rng.integers(0, 2 ** 32, (cols, ncols + 2), dtype=np.uint32)
        terms.append((rr, cols, to_dev_ring(D)[:, 1: 1 + ncols]))
        prod = ring_matmul(P, D[:, 1: 1 + ncols])
        want = ring_sub(want, prod) if subtract else ring_add(want, prod)
    m.mosaic_sparse_stream_gather_rows_terms(terms, rows, ncols, c[:, 1: 1 + ncols], subtract=subtract)
    got = to_np_u32(c)
    assert np.array_equal(got[:, 1: 1 + ncols], want)
    assert np.all(got[:, 0] == 7) and np.all(got[:, 1 + ncols:] == 7)


@pytest.mark.parametrize("name", list(LEVELS))
@pytest.mark.parametrize("M,N", [(1, 33), (2, 100), (3, 31), (4, 64), (5, 1), (8, 8193), (17, 130)])
def test_gather_cols_terms(name, M, N):
    rng = np.random.default_rng(M * 13 + N)
    terms, want = [], rng.integers(0, 2 ** 32, (M, N), dtype=np.uint32)
    c = to_dev_ring(want)
    for rr, cols, P in _levels(name, N):
        D = rng.integers(0, 2 ** 32, (M, cols + 3), dtype=np.uint32)
        terms.append((m.mosaic_sparse_csr(rr, N, cols), to_dev_ring(D)[:, 2: 2 + cols]))
        want = ring_sub(want, ring_matmul(D[:, 2: 2 + cols], P.T))
    sr, sc = torch.rand(M, device="cuda") * 1e-3, torch.rand(N, device="cuda") * 1e-3
    bias = torch.randn(N, device="cuda")
    y = torch.empty((M, N), device="cuda")
    m.mosaic_sparse_gather_cols_terms(terms, M, c, subtract=True, y_f32=y, s_rows=sr, s_cols=sc, bias=bias)
    assert np.array_equal(to_np_u32(c), want)
    ref = (want.view(np.int32).astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
    assert np.array_equal(y.cpu().numpy(), (ref + bias.cpu().numpy()[None, :]).astype(np.float32))


@pytest.mark.parametrize("M", [1, 3, 8, 17])
@pytest.mark.parametrize("stride", [0, 7])
def test_gather_cols_terms_rows_that_overlap(M, stride):
    """d as a view whose rows share memory, against the same matrix laid out in
    full, staged in LDS and (wide rows) gathered from memory."""
    rng = np.random.default_rng(M + stride)
    N = 40
    for cols in (64, 21000):
        flat = to_dev_ring(rng.integers(0, 2 ** 32, (1, cols + stride * M), dtype=np.uint32))[0]
        d = flat.as_strided((M, cols), (stride, 1))
        p = m.mosaic_sparse_csr(m.rng(8, 0x61, 3, m.DIST_SPARSE, log2_inv_density=3), N, cols)
        got, want = (torch.zeros((M, N), dtype=torch.int32, device="cuda") for _ in range(2))
        m.mosaic_sparse_gather_cols_terms([(p, d)], M, got)
        m.mosaic_sparse_gather_cols(p, d.contiguous(), M, want)
        assert torch.equal(got, want)


def test_gather_cols_more_rows_than_a_launch_has_threads():
    """2^23 rows of d and more go in several launches, in the single gather too."""
    M, N, cols = 2 ** 24 + 9, 2, 600
    p = m.mosaic_sparse_csr(m.rng(8, 0x61, 3, m.DIST_SPARSE, log2_inv_density=3), N, cols)
    row = to_dev_ring(np.random.default_rng(4).integers(0, 2 ** 32, (1, cols + 8), dtype=np.uint32))[0]
    d = row.as_strided((M, cols), (0, 1))
    want = torch.zeros((1, N), dtype=torch.int32, device="cuda")
    m.mosaic_sparse_gather_cols(p, d[:1], 1, want)
    for call in (lambda c: m.mosaic_sparse_gather_cols_terms([(p, d)], M, c), lambda c: m.mosaic_sparse_gather_cols(p, d, M, c)):
        c = torch.zeros((M, N), dtype=torch.int32, device="cuda")
        call(c)
        assert torch.equal(c, want.expand(M, N))


@pytest.mark.parametrize("levels", [1, 2])
def test_gather_cols_terms_of_few_entries(levels):
    """Four entries per row of 1536 columns: the single gathers run, the last one
    with the dequantised output, against the oracle."""
    from tests.dispatch_util import gather_cols_sparse
    M, N, cols, t = 18, 4000, 1536, 4
    assert gather_cols_sparse(levels, M, N, levels * cols, levels * t)
    rng = np.random.default_rng(levels)
    want = rng.integers(0, 2 ** 32, (M, N), dtype=np.uint32)
    c, terms = to_dev_ring(want), []
    for k in range(levels):
        D = rng.integers(0, 2 ** 32, (M, cols + 3), dtype=np.uint32)
        P = smp.sample_matrix("weight", N, cols, 8, 0x60 + k, 3, row_weight=t)
        terms.append((m.mosaic_sparse_csr(m.rng(8, 0x60 + k, 3, m.DIST_WEIGHT, row_weight=t), N, cols),
                      to_dev_ring(D)[:, 2: 2 + cols]))
        want = ring_sub(want, ring_matmul(D[:, 2: 2 + cols], P.T))
    sr, sc = torch.rand(M, device="cuda") * 1e-3, torch.rand(N, device="cuda") * 1e-3
    before = c.clone()
    for bad in (dict(bias=sc), dict(y_f32=torch.empty((1, N), device="cuda").expand(M, N), s_rows=sr, s_cols=sc)):
        with pytest.raises(m.MosaicError):       # refused before anything is added
            m.mosaic_sparse_gather_cols_terms(terms, M, c, **bad)
        assert torch.equal(c, before)
    y = torch.empty((M, N), device="cuda")
    m.mosaic_sparse_gather_cols_terms(terms, M, c, subtract=True, y_f32=y, s_rows=sr, s_cols=sc)
    assert np.array_equal(to_np_u32(c), want)
    ref = (want.view(np.int32).astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
    assert np.array_equal(y.cpu().numpy(), ref)
