"""Mask pass and row quantisation on rows of any length at any element
address: row lengths around the lane (4 columns), the digit group (16), the
workgroup (1024 columns) and the register-resident sizes, with bases and
pitches that are not multiples of 16 bytes. Every output bit equals the
oracle's, and nothing outside the rows is written."""
import numpy as np
import pytest
import torch

from tests.gpu_util import pad_is_zero, to_dev_ring, to_np_u32, unpack_digits

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_29221_amd import mosaic as m
    from paper_2607_29221_amd.mosaic import Digits

KINDS = {"uniform": 1, "dgauss": 2, "sparse": 3}


@pytest.mark.parametrize("cols", [1, 3, 5, 17, 63, 66, 1021, 1023, 1025, 2047, 4099])
@pytest.mark.parametrize("kind", [None, "uniform", "dgauss", "sparse"])
@pytest.mark.parametrize("dtype", ["none", "int8", "int16", "int32"])
def test_mask_ragged(cols, kind, dtype):
    from oracle import sampling as smp
    rows, off = 6, 1 + cols % 3
    rng = np.random.default_rng(cols * 7 + len(dtype))
    x = None
    if dtype != "none":
        info = np.iinfo(dtype)
        x = rng.integers(info.min, info.max + 1, (rows, cols + 3)).astype(dtype)
    u = rng.integers(0, 2 ** 32, (rows, cols + 3), dtype=np.uint32)
    noise = None if kind is None else m.rng(91, 0x51, cols, KINDS[kind], sigma=0.5, bound=4, log2_inv_density=2)
    want = u[:, off: off + cols].astype(np.int64) if (x is None or cols % 2) else np.zeros((rows, cols), np.int64)
    with_u = x is None or cols % 2
    if x is not None:
        want = want + x[:, off: off + cols].astype(np.int64)
    if kind is not None:
        want = want + smp.sample_matrix(kind, rows, cols, 91, 0x51, cols, sigma=0.5, bound=4,
                                        log2_inv_density=2).astype(np.int64)
    want = (want & 0xFFFFFFFF).astype(np.uint32)
    out = torch.full((rows, cols + 5), 77, dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, cols)
    m.mosaic_mask(None if x is None else torch.from_numpy(x).cuda()[:, off: off + cols],
                  to_dev_ring(u)[:, off: off + cols] if with_u else None, noise, rows, cols,
                  out=out[:, off: off + cols], out_dig=dig)
    got = to_np_u32(out)
    assert np.array_equal(got[:, off: off + cols], want)
    assert np.all(got[:, :off] == 77) and np.all(got[:, off + cols:] == 77)
    assert np.array_equal(unpack_digits(dig), want) and pad_is_zero(dig)


@pytest.mark.parametrize("n", [1, 2, 7, 1023, 1025, 2050, 4097, 8189, 16385, 32769, 65535, 65538, 70001])
@pytest.mark.parametrize("offset", [0, 1, 2])
def test_quantize_ragged(n, offset):
    from oracle import quant as oquant
    rng = np.random.default_rng(n)
    x = (rng.standard_normal((3, n)) * np.exp(rng.uniform(-9, 9, (3, 1)))).astype(np.float32)
    wide = torch.full((3, n + 3), 1e30, dtype=torch.float32, device="cuda")   # neighbours must not be read as columns
    wide[:, offset: offset + n] = torch.from_numpy(x).cuda()
    q = torch.full((3, n + 3), 77, dtype=torch.int32, device="cuda")
    dig = Digits.empty(3, n)
    sc = torch.empty(3, dtype=torch.float32, device="cuda")
    m.mosaic_quantize_rows(wide[:, offset: offset + n], 1997, q=q[:, offset: offset + n], q_dig=dig, scale=sc)
    qr, sr = oquant.quantize_rows(x, 1997)
    got = q.cpu().numpy()
    assert np.array_equal(sc.cpu().numpy(), sr)
    assert np.array_equal(got[:, offset: offset + n], qr)
    assert np.all(got[:, :offset] == 77) and np.all(got[:, offset + n:] == 77)
    assert np.array_equal(unpack_digits(dig), qr.view(np.uint32)) and pad_is_zero(dig)


@pytest.mark.parametrize("rows,cols", [(1, 9), (3, 65), (64, 64), (63, 130), (66, 1), (130, 67), (257, 300)])
@pytest.mark.parametrize("kind", [None, "uniform", "dgauss", "sparse"])
@pytest.mark.parametrize("dtype", ["none", "int8", "int16", "int32"])
def test_mask_transposed(rows, cols, kind, dtype):
    """Plaintext stored transposed and noise of the transposed matrix, at tile
    edges (64 x 64), row counts that are not multiples of 4 and offsets."""
    from oracle import sampling as smp
    if dtype == "none" and kind is None:
        pytest.skip("neither plaintext nor noise")
    rng = np.random.default_rng(rows * 31 + cols)
    want = np.zeros((rows, cols), np.int64)
    x = None
    if dtype != "none":
        info = np.iinfo(dtype)
        x = rng.integers(info.min, info.max + 1, (cols, rows + 3)).astype(dtype)
        want = want + x[:, 1: 1 + rows].T.astype(np.int64)
    u = rng.integers(0, 2 ** 32, (rows, cols + 1), dtype=np.uint32) if cols % 2 else None
    if u is not None:
        want = want + u[:, 1:].astype(np.int64)
    noise = None
    if kind is not None:
        noise = m.rng(17, 0x31, 2, KINDS[kind], sigma=0.5, bound=4, log2_inv_density=2, transposed=True)
        want = want + smp.sample_matrix(kind, cols, rows, 17, 0x31, 2, sigma=0.5, bound=4,
                                        log2_inv_density=2).T.astype(np.int64)
    want = (want & 0xFFFFFFFF).astype(np.uint32)
    out = torch.full((rows, cols + 2), 77, dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, cols)
    m.mosaic_mask(None if x is None else torch.from_numpy(x).cuda()[:, 1: 1 + rows],
                  None if u is None else to_dev_ring(u)[:, 1:], noise, rows, cols,
                  out=out[:, 1: 1 + cols], out_dig=dig, x_transposed=x is not None)
    got = to_np_u32(out)
    assert np.array_equal(got[:, 1: 1 + cols], want)
    assert np.all(got[:, 0] == 77) and np.all(got[:, 1 + cols:] == 77)
    assert np.array_equal(unpack_digits(dig), want) and pad_is_zero(dig)


def test_mask_more_rows_than_a_launch_has_workgroups():
    """2^24 rows and more: a workgroup per row would pass the launch limit of
    2^32 threads (and run the first few rows alone), for ragged and for aligned
    rows."""
    for cols in (3, 4):
        rows = 2 ** 24 + 5
        x = torch.arange(rows * cols, dtype=torch.int32, device="cuda").reshape(rows, cols)
        out = torch.empty_like(x)
        m.mosaic_mask(x, x, None, rows, cols, out=out)
        assert torch.equal(out, 2 * x)


@pytest.mark.parametrize("rows,cols", [(2049, 3), (6145, 17), (6144, 18)])
@pytest.mark.parametrize("kind", ["uniform", "dgauss", "sparse"])
def test_mask_many_short_rows(rows, cols, kind):
    """Either side of the row count from which short ragged rows take the
    general kernel."""
    from oracle import sampling as smp
    rng = np.random.default_rng(cols)
    x = rng.integers(-2 ** 15, 2 ** 15, (rows, cols + 1)).astype(np.int16)
    u = rng.integers(0, 2 ** 32, (rows, cols + 1), dtype=np.uint32)
    e = smp.sample_matrix(kind, rows, cols, 91, 0x51, cols, sigma=0.5, bound=4, log2_inv_density=2)
    want = ((x[:, 1:].astype(np.int64) + u[:, 1:] + e.astype(np.int64)) & 0xFFFFFFFF).astype(np.uint32)
    out = torch.full((rows, cols + 2), 77, dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, cols)
    m.mosaic_mask(torch.from_numpy(x).cuda()[:, 1:], to_dev_ring(u)[:, 1:],
                  m.rng(91, 0x51, cols, KINDS[kind], sigma=0.5, bound=4, log2_inv_density=2), rows, cols,
                  out=out[:, 1: 1 + cols], out_dig=dig)
    got = to_np_u32(out)
    assert np.array_equal(got[:, 1: 1 + cols], want)
    assert np.all(got[:, 0] == 77) and np.all(got[:, 1 + cols:] == 77)
    assert np.array_equal(unpack_digits(dig), want) and pad_is_zero(dig)


@pytest.mark.parametrize("n", [3, 4])
def test_quantize_more_rows_than_a_launch_has_workgroups(n):
    """The codes, digits and scales of 2^24 rows and more are those of their parts."""
    rows, cut = 2 ** 24 + 5, 2 ** 21 + 1
    x = torch.empty((rows, n), device="cuda").normal_()
    q, sc = torch.zeros((rows, n), dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda")
    m.mosaic_quantize_rows(x, 1997, q=q, scale=sc)
    for r in range(0, rows, cut):
        k = min(cut, rows - r)
        qp, sp = torch.empty((k, n), dtype=torch.int32, device="cuda"), torch.empty(k, device="cuda")
        m.mosaic_quantize_rows(x[r: r + k], 1997, q=qp, scale=sp)
        assert torch.equal(q[r: r + k], qp) and torch.equal(sc[r: r + k], sp)
