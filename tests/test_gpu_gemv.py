"""Products of one and two rows by dot products, at the edges of their steps
(256 columns), of the loads fetched ahead (1024), of a wave's and a
workgroup's rows of B (2 and 8) and of the rule that selects them (2048
columns for two rows, 6144 for one), against the oracle."""
import numpy as np
import pytest
import torch

from tests.gpu_util import to_dev_ring, to_np_u32

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_29221_amd import mosaic as m
    from paper_2607_29221_amd.mosaic import Digits


def _ring(rng, shape):
    """Ring words, some rows of the largest digit magnitudes (-128 and 127)."""
    x = rng.integers(0, 2 ** 32, shape, dtype=np.uint32)
    x[::3] = rng.choice(np.array([0x7F7F7F80, 0x7F7F7F7F, 0x80808080, 0xFFFFFFFF, 0], dtype=np.uint32),
                        x[::3].shape)
    return x


def _digits(x, col0=0):
    """Digits of x in a buffer with 64 columns of other digits on either side."""
    rows, cols = x.shape
    buf = torch.randint(-128, 128, (rows, 4 * (col0 + m.padded_k(cols) + 64)), device="cuda", dtype=torch.int8)
    d = Digits(buf, cols, col0)
    m.mosaic_mask(None, to_dev_ring(x), None, rows, cols, out_dig=d)
    return d


SIZES = [(1, N, K) for N in (1, 2, 7, 9, 257) for K in (1, 64, 100, 256, 260, 1024, 1088, 3000)]
SIZES += [(1, 1025, 4096), (1, 3073, 6144), (1, 70, 6144), (1, 70, 6208), (2, 1, 64), (2, 9, 260), (2, 130, 1028), (2, 33, 2048), (2, 33, 2112)]


@pytest.mark.parametrize("M,N,K", SIZES)
def test_product_and_unmask(M, N, K):
    from oracle.ring import ring_matmul
    rng = np.random.default_rng(7 * M + N + K)
    a, b = _ring(rng, (M, K)), _ring(rng, (N, K))
    want = ring_matmul(a, np.ascontiguousarray(b.T))
    B = _digits(b, 64)
    c = torch.full((M + 1, N + 3), 5, dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(_digits(a, 128), B, M, N, K, c[:M, :N])
    got = to_np_u32(c)
    assert np.array_equal(got[:M, :N], want)
    assert np.all(got[:, N:] == 5) and np.all(got[M] == 5)

    # Q as ring words with other words after its columns
    pad = -K % 4
    q = to_dev_ring(np.concatenate([a, rng.integers(0, 2 ** 32, (M, pad + 8), dtype=np.uint32)], axis=1))[:, :K]
    ym, kc = _ring(rng, (M, N)), _ring(rng, (M, N))
    y = torch.full((M + 1, N + 3), 5, dtype=torch.int32, device="cuda")
    sr, sc = torch.rand(M, device="cuda"), torch.rand(N, device="cuda")
    bias, f = torch.rand(N, device="cuda"), torch.empty((M, N), device="cuda")
    m.mosaic_unmask_words(to_dev_ring(ym), to_dev_ring(kc), q, B, M, N, K, y=y[:M, :N], s_rows=sr, s_cols=sc,
                          y_f32=f, bias=bias)
    out = ym - kc - want
    got = to_np_u32(y)
    assert np.array_equal(got[:M, :N], out)
    assert np.all(got[:, N:] == 5) and np.all(got[M] == 5)
    ref = out.view(np.int32).astype(np.float32) * sr.cpu().numpy()[:, None] * sc.cpu().numpy() + bias.cpu().numpy()
    assert np.array_equal(f.cpu().numpy(), ref)

    # in place, without K_c
    t = to_dev_ring(ym)
    m.mosaic_unmask_words(t, None, q, B, M, N, K, y=t)
    assert np.array_equal(to_np_u32(t), ym - want)
