"""The forms of the tiled ring product (64-row tiles with the stages split
between two groups of waves, 64-row tiles two workgroups to a compute unit,
128-row tiles whole and split along K) at tile edges and at every kind of
stage count: one stage per group, odd shares, and counts around the steady
loop's period. Products against the oracle, and against the short-A kernel in
row slices where the matrices are large."""
import numpy as np
import pytest
import torch

from tests.dispatch_util import gemm_plan
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


def _plan(M, N, K, epilogue):
    return gemm_plan(M, N, K, epilogue, torch.cuda.get_device_properties(0).multi_processor_count)


def _random_digits(M, K, g):
    return Digits(torch.randint(-128, 128, (M, 4 * m.padded_k(K)), generator=g, device="cuda", dtype=torch.int8), K)


def _by_slices(A, B, M, N, K):
    """The product by the short-A kernel, 64 rows at a time."""
    want = torch.empty((M, N), dtype=torch.int32, device="cuda")
    for r0 in range(0, M, 64):
        rows = min(64, M - r0)
        m.mosaic_masked_matmul(Digits(A.buf[r0: r0 + rows], K), B, rows, N, K, want[r0: r0 + rows])
    return want


def _ref(a, b):
    from oracle.ring import ring_matmul
    return ring_matmul(a, np.ascontiguousarray(b.T))


@pytest.mark.parametrize("M,N", [(65, 1), (65, 130), (128, 128), (129, 257), (200, 127)])
@pytest.mark.parametrize("K", [1, 64, 128, 192, 320, 384, 448, 512, 576, 768, 832])
def test_few_tiles(M, N, K):
    assert _plan(M, N, K, "store")[0] == _plan(M, N, K, "unmask")[0] == "64k"
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


@pytest.mark.parametrize("M,N,K,form", [
    (257, 11005, 192, "64"), (257, 11008, 1536, "64"), (385, 11264, 704, "64"), (513, 8704, 64, "64"),
    (130, 9728, 2048, "64k"), (66, 9729, 4160, "64k")])
def test_many_tiles(M, N, K, form):
    """Tile counts of one and a bit rounds of the chip (64-row tiles two to a
    unit) and of part of a round (their stages between two groups of waves; the
    store of the last one takes 128-row tiles split along K)."""
    assert _plan(M, N, K, "unmask")[0] == form
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    A, B = _random_digits(M, K, g), _random_digits(N, K, g)
    want = _by_slices(A, B, M, N, K)
    c = torch.full((M, N), 5, dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, K, c)
    assert torch.equal(c, want)
    ym = torch.randint(-2 ** 31, 2 ** 31, (M, N), generator=g, device="cuda", dtype=torch.int32)
    y = torch.full((M, N), 5, dtype=torch.int32, device="cuda")
    m.mosaic_unmask(ym, None, A, B, M, N, K, y=y)
    assert torch.equal(y, ym - want)


# 4096 columns of K: 128 stages, the others the stage counts 6, 8, 10, 14 and 16 at
# eight rounds of 128-row tiles, from which no other form is chosen
WHOLE_128 = [(333, 9731, 4096)] + [(1100, 29201, K) for K in (192, 256, 320, 448, 512)] + [(2000, 1100, 512)]


@pytest.mark.parametrize("M,N,K", WHOLE_128)
def test_whole_128_row_tiles(M, N, K):
    """128-row tiles whole: stored to a window of a wider matrix and unmasked in
    place on Y' and on K_c and to floats, with widths, pitches and bases that are
    not multiples of 16 bytes (1100 columns: all of them are)."""
    assert _plan(M, N, K, "store") == _plan(M, N, K, "unmask") == ("128", 0, 1)
    off = N % 4
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K)
    A, B = _random_digits(M, K, g), _random_digits(N, K, g)
    want = _by_slices(A, B, M, N, K)

    def window():
        return torch.randint(-2 ** 31, 2 ** 31, (M, N + 4 * off), generator=g, device="cuda", dtype=torch.int32)

    def outside(t, before):
        return torch.equal(t[:, :off], before[:, :off]) and torch.equal(t[:, off + N:], before[:, off + N:])

    c = window()
    before = c.clone()
    m.mosaic_masked_matmul(A, B, M, N, K, c[:, off: off + N])
    assert torch.equal(c[:, off: off + N], want) and outside(c, before)
    del c, before
    ym, kc = window(), window()
    ref = ym[:, off: off + N] - kc[:, off: off + N] - want
    del want
    f = torch.empty((M, N), device="cuda")
    sr, sc = torch.rand(M, device="cuda"), torch.rand(N + 3, device="cuda")[off: off + N]
    bias = torch.randn(N + 3, device="cuda")[off: off + N]
    m.mosaic_unmask(ym[:, off: off + N], kc[:, off: off + N], A, B, M, N, K, s_rows=sr, s_cols=sc, y_f32=f, bias=bias)
    assert torch.equal(f, ref.float() * sr[:, None] * sc[None, :] + bias[None, :])
    for t in (0, 1):
        ops = [ym.clone(), kc.clone()]
        m.mosaic_unmask(ops[0][:, off: off + N], ops[1][:, off: off + N], A, B, M, N, K, y=ops[t][:, off: off + N])
        assert torch.equal(ops[t][:, off: off + N], ref) and outside(ops[t], (ym, kc)[t])
        assert torch.equal(ops[1 - t], (ym, kc)[1 - t])


@pytest.mark.parametrize("M,N,K,split", [(66, 9729, 4160, (77, 3)), (130, 4099, 4160, (66, 3)), (200, 16387, 4160, (2, 8)),
                                         (66, 4099, 4160, (33, 6))])
@pytest.mark.parametrize("accumulate", [False, True])
def test_split_128_row_tiles(M, N, K, split, accumulate):
    """The last round's tiles in pieces along K, as a store (cleared first) and as
    the second chunk of a longer K, which is added into what the first stored."""
    long_k = 32704 + K if accumulate else K
    assert _plan(M, N, K, "accum" if accumulate else "store") == ("128",) + split
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N)
    A, B = _random_digits(M, long_k, g), _random_digits(N, long_k, g)
    c = torch.full((M, N + 5), 7, dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, long_k, c[:, 3: 3 + N])
    assert torch.equal(c[:, 3: 3 + N], _by_slices(A, B, M, N, long_k))
    assert torch.all(c[:, :3] == 7) and torch.all(c[:, 3 + N:] == 7)


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
