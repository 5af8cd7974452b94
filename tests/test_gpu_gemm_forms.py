"""The forms of the tiled ring product (64-row tiles with the stages split
between two groups of waves, 64-row tiles two workgroups to a compute unit,
128-row tiles whole and split along K) at tile edges and at every kind of
stage count: one stage per group, odd shares, and counts around the steady
loop's period. Products against the oracle, and against the short-A kernel in
row slices where the matrices are large."""
import numpy as np
import pytest
import torch

from tests.gpu_util import to_dev_ring, to_np_u32

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_29221_amd import mosaic as m
    from paper_2607_29221_amd.mosaic import Digits


def _digits(x):
    d = Digits.empty(*x.shape)
    m.mosaic_mask(None, to_dev_ring(x), None, x.shape[0], x.shape[1], out_dig=d)
    return d


def _ring(rng, shape):
    return rng.integers(0, 2 ** 32, shape, dtype=np.uint32)


def _ref(a, b):
    from oracle.ring import ring_matmul
    return ring_matmul(a, np.ascontiguousarray(b.T))


@pytest.mark.parametrize("M,N", [(65, 1), (65, 130), (128, 128), (129, 257), (200, 127)])
@pytest.mark.parametrize("K", [1, 64, 128, 192, 320, 384, 448, 512, 576, 768, 832])
def test_few_tiles(M, N, K):
    rng = np.random.default_rng(M + N + K)
    a, b = _ring(rng, (M, K)), _ring(rng, (N, K))
    c = torch.full((M, N + 3), 5, dtype=torch.int32, device="cuda")
    A, B = _digits(a), _digits(b)
    m.mosaic_masked_matmul(A, B, M, N, K, c[:, :N])
    want = _ref(a, b)
    got = to_np_u32(c)
    assert np.array_equal(got[:, :N], want)
    assert np.all(got[:, N:] == 5)
    ym, kc = _ring(rng, (M, N)), _ring(rng, (M, N))
    y = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_unmask(to_dev_ring(ym), to_dev_ring(kc), A, B, M, N, K, y=y)
    assert np.array_equal(to_np_u32(y), ym - kc - want)


@pytest.mark.parametrize("M,N,K", [(257, 11005, 192), (257, 11008, 1536), (385, 11264, 704), (513, 8704, 64),
                                   (130, 9728, 2048), (66, 9729, 4160)])
def test_many_tiles(M, N, K):
    """Tile counts of one and a bit rounds of the chip (64-row tiles two to a
    unit) and partial rounds (split along K)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    A = Digits(torch.randint(-128, 128, (M, 4 * m.padded_k(K)), generator=g, device="cuda", dtype=torch.int8), K)
    B = Digits(torch.randint(-128, 128, (N, 4 * m.padded_k(K)), generator=g, device="cuda", dtype=torch.int8), K)
    want = torch.empty((M, N), dtype=torch.int32, device="cuda")
    for r0 in range(0, M, 64):
        rows = min(64, M - r0)
        m.mosaic_masked_matmul(Digits(A.buf[r0: r0 + rows], K), B, rows, N, K, want[r0: r0 + rows])
    c = torch.full((M, N), 5, dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, K, c)
    assert torch.equal(c, want)
    ym = torch.randint(-2 ** 31, 2 ** 31, (M, N), generator=g, device="cuda", dtype=torch.int32)
    y = torch.full((M, N), 5, dtype=torch.int32, device="cuda")
    m.mosaic_unmask(ym, None, A, B, M, N, K, y=y)
    assert torch.equal(y, ym - want)


@pytest.mark.parametrize("M", [3, 8, 9, 16])
@pytest.mark.parametrize("N", [4096, 4097, 12288, 12289])
@pytest.mark.parametrize("K", [64, 192, 704])
def test_unmask_words_forms(M, N, K):
    """The forms of the unmask with Q as ring words at the column counts where
    they change (16 and 48 per compute unit of 256), with fewer stages than
    waves and shares that differ."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    q = torch.randint(-2 ** 31, 2 ** 31, (M, K), generator=g, device="cuda", dtype=torch.int32)
    A = Digits.empty(M, K)
    m.mosaic_mask(None, q, None, M, K, out_dig=A)
    B = Digits(torch.randint(-128, 128, (N, 4 * m.padded_k(K)), generator=g, device="cuda", dtype=torch.int8), K)
    prod = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, K, prod)
    ym = torch.randint(-2 ** 31, 2 ** 31, (M, N), generator=g, device="cuda", dtype=torch.int32)
    y = torch.full((M, N + 1), 5, dtype=torch.int32, device="cuda")
    m.mosaic_unmask_words(ym, None, q, B, M, N, K, y=y[:, :N])
    assert torch.equal(y[:, :N], ym - prod)
    assert torch.all(y[:, N] == 5)


@pytest.mark.parametrize("M,N,K", [(8, 8192, 1088), (8, 8193, 1088), (16, 12289, 3136), (1, 12289, 6208)])
def test_unmask_words_long_inner(M, N, K):
    """Either side of the inner dimensions where those forms change."""
    test_unmask_words_forms(M, N, K)
