"""The rotation of short blocks (several to a workgroup) and of the longest
ones (1024 threads each), and the fused input pass of the row lengths that one
launch holds in registers: against the float64 oracle and, bit for bit, the
separate passes."""
import numpy as np
import pytest
import torch

from oracle import hadamard as ohad
from oracle import sampling as smp
from tests.gpu_util import digits_np

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_29221_amd import mosaic as m
    from paper_2607_29221_amd.mosaic import Digits


@pytest.mark.parametrize("b", [16, 32, 64, 128, 16384, 32768])
@pytest.mark.parametrize("rows,blocks,pad", [(1, 1, 0), (3, 1, 4), (70, 3, 0), (33, 7, 8), (129, 13, 4)])
@pytest.mark.parametrize("inverse", [False, True])
def test_rotation(b, rows, blocks, pad, inverse):
    if b >= 16384:
        rows, blocks = min(rows, 5), min(blocks, 2)
    n = b * blocks
    rng = np.random.default_rng(b + rows)
    x = rng.standard_normal((rows, n)).astype(np.float32)
    x[0, n // 2] *= 50.0
    signs = smp.sample_signs(n, 5, 1)
    wide = torch.zeros((rows, n + pad), device="cuda")
    wide[:, :n] = torch.from_numpy(x).cuda()
    y = torch.full((rows, n + 2 * pad), 7.0, device="cuda")
    m.mosaic_hadamard_rotate(wide[:, :n], y[:, :n], block=b, signs=torch.from_numpy(signs).cuda(), inverse=inverse)
    ref = ohad.rotate(x.astype(np.float64), signs, block=b, inverse=inverse)
    got = y.cpu().numpy()
    err = np.max(np.abs(got[:, :n] - ref), axis=1) / np.max(np.abs(ref), axis=1)
    assert np.all(err <= 1e-5)
    assert np.all(got[:, n:] == 7.0)
    m.mosaic_hadamard_rotate(wide[:, :n], wide[:, :n], block=b, signs=torch.from_numpy(signs).cuda(), inverse=inverse)
    assert np.array_equal(wide.cpu().numpy()[:, :n], got[:, :n])          # in place: the same bits


@pytest.mark.parametrize("block,count", [(1024, c) for c in (1, 2, 3, 5, 7, 8, 9, 10, 11)]
                         + [(2048, c) for c in (1, 3, 5, 7)] + [(4096, c) for c in (1, 2, 3)] + [(8192, 1), (16384, 1),
                                                                                              (16384, 2)])
@pytest.mark.parametrize("noise", [None, "dgauss", "uniform", "sparse"])
def test_fused_rows(block, count, noise):
    rows, n, qmax = 3, block * count, 567
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn((rows, n), generator=g, device="cuda")
    x[0, 5] *= 50
    x[1] = 0.0
    signs = torch.empty(n, dtype=torch.int8, device="cuda")
    m.mosaic_sample_signs(m.rng(17, 0x70, 2, 0), n, signs)
    u = torch.randint(-2 ** 31, 2 ** 31, (rows, n + 4), generator=g, device="cuda", dtype=torch.int32)[:, :n]
    kinds = {"uniform": m.DIST_UNIFORM, "dgauss": m.DIST_DGAUSS, "sparse": m.DIST_SPARSE}
    nz = None if noise is None else m.rng(19, 0x50, 4, kinds[noise], sigma=1.7, bound=6, log2_inv_density=2)
    y, q = torch.empty_like(x), torch.empty((rows, n), dtype=torch.int32, device="cuda")
    s_ref, s = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    d_ref, d = Digits.empty(rows, n), Digits.empty(rows, n)
    m.mosaic_hadamard_rotate(x, y, block=block, signs=signs)
    m.mosaic_quantize_rows(y, qmax, q=q, scale=s_ref)
    m.mosaic_mask(q, u, nz, rows, n, out_dig=d_ref)
    m.mosaic_rotate_quantize_mask(x, qmax, d, block=block, signs=signs, u=u, noise=nz, scale=s)
    assert torch.equal(s, s_ref)
    assert np.array_equal(digits_np(d), digits_np(d_ref))
