"""Parity of each HIP entry point with the CPU oracle on seeded inputs that
span several tiles and ragged tails. Ring results must match bit for bit; the
rotation to 1e-5 of each row's peak (fp32 against the float64 oracle)."""
import numpy as np
import pytest
import torch

from oracle import hadamard as ohad
from oracle import quant as oquant
from oracle import sampling as smp
from oracle.ring import ring_matmul, ring_sub, signed_digits
from paper_2607_29221_amd import mosaic as m
from paper_2607_29221_amd.mosaic import Digits
from tests.gpu_util import pad_is_zero, to_dev_ring, to_np_u32, unpack_digits

pytestmark = pytest.mark.gpu

SEED = 0x5EED_0001_2345_6789


def _rng_np(seed):
    return np.random.default_rng(seed)


@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 37), (64, 512), (33, 130)])
@pytest.mark.parametrize("kind", ["uniform", "dgauss", "sparse"])
@pytest.mark.parametrize("transposed", [False, True])
def test_sample(rows, cols, kind, transposed):
    dist = {"uniform": m.DIST_UNIFORM, "dgauss": m.DIST_DGAUSS, "sparse": m.DIST_SPARSE}[kind]
    r = m.rng(SEED, 0x33, 7, dist, sigma=0.5, bound=4, log2_inv_density=2, transposed=transposed)
    out = torch.empty((rows, cols), dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, cols)
    m.mosaic_sample(r, rows, cols, out=out, out_dig=dig)
    torch.cuda.synchronize()
    if transposed:
        ref = smp.sample_matrix(kind, cols, rows, SEED, 0x33, 7, sigma=0.5, bound=4, log2_inv_density=2).T
    else:
        ref = smp.sample_matrix(kind, rows, cols, SEED, 0x33, 7, sigma=0.5, bound=4, log2_inv_density=2)
    assert np.array_equal(to_np_u32(out), ref)
    assert np.array_equal(unpack_digits(dig), ref)
    assert pad_is_zero(dig)


def test_digit_bytes_are_balanced_digits():
    x = _rng_np(1).integers(0, 2 ** 32, (3, 80), dtype=np.uint64).astype(np.uint32)
    x[0, :8] = [0, 1, 0x7F, 0x80, 0xFF, 0x80808080, 0x7F7F7F80, 0xFFFFFFFF]
    dig = Digits.empty(3, 80)
    m.mosaic_mask(to_dev_ring(x), None, None, 3, 80, out_dig=dig)
    raw = dig.buf.cpu().numpy().reshape(3, 128 // 16, 4, 16)
    d = signed_digits(x)                          # (3, 80, 4)
    for k in range(80):
        g, b = divmod(k, 16)
        assert np.array_equal(raw[:, g, :, b], d[:, k, :])


def test_signs():
    for n in (1, 7, 8192, 28672):
        out = torch.empty(n, dtype=torch.int8, device="cuda")
        m.mosaic_sample_signs(m.rng(SEED, 0x70, 3, 0), n, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), smp.sample_signs(n, SEED, 3))


@pytest.mark.parametrize("dtype", [torch.int8, torch.int16, torch.int32])
@pytest.mark.parametrize("rows,cols", [(7, 100), (64, 512), (2, 16), (3, 70)])
@pytest.mark.parametrize("u_pad", [3, 4])
def test_mask(dtype, rows, cols, u_pad):
    rng = _rng_np(rows * cols)
    info = {torch.int8: (-128, 128), torch.int16: (-32768, 32768), torch.int32: (-2 ** 31, 2 ** 31)}[dtype]
    x = rng.integers(info[0], info[1], (rows, cols)).astype({torch.int8: np.int8, torch.int16: np.int16,
                                                             torch.int32: np.int32}[dtype])
    u = rng.integers(0, 2 ** 32, (rows, cols + u_pad), dtype=np.uint64).astype(np.uint32)
    noise = m.rng(SEED, 0x50, 9, m.DIST_DGAUSS, sigma=0.5, bound=4)
    out = torch.empty((rows, cols), dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, cols)
    u_dev = to_dev_ring(u)
    m.mosaic_mask(torch.from_numpy(x).cuda(), u_dev[:, :cols], noise, rows, cols, out=out, out_dig=dig)
    torch.cuda.synchronize()
    e = smp.sample_matrix("dgauss", rows, cols, SEED, 0x50, 9)
    ref = ((x.astype(np.int64) & 0xFFFFFFFF) + u[:, :cols].astype(np.int64) + e.astype(np.int64)) & 0xFFFFFFFF
    assert np.array_equal(to_np_u32(out), ref.astype(np.uint32))
    assert np.array_equal(unpack_digits(dig), ref.astype(np.uint32))


def test_mask_transposed_input_and_sparse_noise():
    rows, cols = 40, 72
    xt = _rng_np(3).integers(-127, 128, (cols, rows)).astype(np.int8)      # stored transposed
    noise = m.rng(SEED, 0x41, 1, m.DIST_SPARSE, log2_inv_density=3)
    dig = Digits.empty(rows, cols)
    m.mosaic_mask(torch.from_numpy(xt).cuda(), None, noise, rows, cols, out_dig=dig, x_transposed=True)
    torch.cuda.synchronize()
    e = smp.sample_matrix("sparse", rows, cols, SEED, 0x41, 1, log2_inv_density=3)
    ref = ((xt.T.astype(np.int64) & 0xFFFFFFFF) + e) & 0xFFFFFFFF
    assert np.array_equal(unpack_digits(dig), ref.astype(np.uint32))


def _random_ring(rng, shape, edge=False):
    x = rng.integers(0, 2 ** 32, shape, dtype=np.uint64).astype(np.uint32)
    if edge:
        flat = x.reshape(-1)
        vals = np.array([0, 1, 0x7FFFFFFF, 0x80000000, 0xFFFFFFFF, 0x80808080, 0x7F7F7F80], dtype=np.uint32)
        flat[: min(flat.size, 64)] = np.resize(vals, min(flat.size, 64))
    return x


def _gemm(a_np, b_np):
    M, K = a_np.shape
    N = b_np.shape[0]
    A, B = Digits.empty(M, K), Digits.empty(N, K)
    m.mosaic_mask(to_dev_ring(a_np), None, None, M, K, out_dig=A)
    m.mosaic_mask(to_dev_ring(b_np), None, None, N, K, out_dig=B)
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, K, C)
    torch.cuda.synchronize()
    return to_np_u32(C)


@pytest.mark.parametrize("M,N,K", [(64, 512, 512), (1, 1, 1), (300, 260, 1000), (130, 129, 70),
                                   (128, 128, 64), (257, 3, 192), (5, 300, 4096), (0, 10, 64), (10, 10, 0)])
def test_masked_matmul(M, N, K):
    rng = _rng_np(M * 7 + N * 3 + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    got = _gemm(a, b)
    assert np.array_equal(got, ring_matmul(a, b.T))


@pytest.mark.parametrize("M,N,K", [(200, 1000, 4096), (130, 3000, 2048), (200, 1001, 4096), (65, 130, 512),
                                   (300, 4099, 640)])
def test_masked_matmul_mid_size(M, N, K):
    """Tiled-kernel products with fewer tiles than compute units and a long
    K range, checked in full: 64-row tiles whose stages two groups of waves
    share, and 128-row tiles in eight pieces along K added atomically after a
    clear of their outputs (K = 4096); N = 1001 and 4099 take the epilogue of
    unaligned rows."""
    rng = _rng_np(M + N + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    assert np.array_equal(_gemm(a, b), ring_matmul(a, b.T))


@pytest.mark.parametrize("K", [192, 256, 288, 320, 448, 512, 1536])
def test_masked_matmul_stage_loop_forms(K):
    """Whole-tile products (144 tiles: one round, no split-K pieces) whose
    32-column stage counts take each form of the stage loop: below eight
    stages the general loop only (K = 192: 6 stages); exactly eight (the
    four-stage loop once, then the last four as straight code); 4 q + 2
    stages (K = 288 and 320: 10, K padded to a multiple of 64; 448: 14),
    whose last six take the general loop; multiples of four (512: 16, 1536:
    48). The last tile is ragged in both dimensions."""
    rng = _rng_np(K + 17)
    M, N = 2000, 1100
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    assert np.array_equal(_gemm(a, b), ring_matmul(a, b.T))


def test_masked_matmul_split_output_window():
    """Split-K pieces writing into a window of a wider C (ldc > N, a column
    offset): the clear before a store and the atomic adds touch only the
    window; K past one launch's range makes the second chunk accumulate, in
    64-row tiles."""
    M, N, K = 150, 203, 33000
    rng = _rng_np(5)
    a = _random_ring(rng, (M, K))
    b = _random_ring(rng, (N, K))
    A, B = Digits.empty(M, K), Digits.empty(N, K)
    m.mosaic_mask(to_dev_ring(a), None, None, M, K, out_dig=A)
    m.mosaic_mask(to_dev_ring(b), None, None, N, K, out_dig=B)
    C0 = _random_ring(rng, (M, N + 9))
    C = to_dev_ring(C0)
    m.mosaic_masked_matmul(A, B, M, N, K, C[:, 3:3 + N])
    torch.cuda.synchronize()
    got = to_np_u32(C)
    assert np.array_equal(got[:, 3:3 + N], ring_matmul(a, b.T))
    assert np.array_equal(got[:, :3], C0[:, :3]) and np.array_equal(got[:, 3 + N:], C0[:, 3 + N:])


@pytest.mark.parametrize("M", [1, 8, 15, 16, 17, 33, 48, 63, 64, 65])
@pytest.mark.parametrize("N,K", [(33, 64), (100, 576), (16, 1000), (47, 4160)])
def test_masked_matmul_short_a(M, N, K):
    """Decode-shaped products (at most 64 rows of A take the shared-A decode
    kernel): row counts on and around the 16-row tiles, ragged N inside one
    128-row column tile, and K ranges of 1 to 65 stages cut into per-workgroup
    ranges whose partial products are added atomically."""
    rng = _rng_np(M * 131 + N * 7 + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    assert np.array_equal(_gemm(a, b), ring_matmul(a, b.T))


@pytest.mark.parametrize("M", [1, 16, 17, 40, 64])
@pytest.mark.parametrize("N,K", [(1000, 4160), (3000, 576), (300, 64), (2049, 1024)])
def test_masked_matmul_short_a_many_tiles(M, N, K):
    """Decode kernel over several 128-row column tiles with a ragged last
    tile: the workgroups' (tile, stage) ranges start and end inside tiles and
    cross tile boundaries (one to a few stages each), or hold single-stage
    tiles (K = 64)."""
    rng = _rng_np(M * 17 + N * 5 + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    assert np.array_equal(_gemm(a, b), ring_matmul(a, b.T))


@pytest.mark.parametrize("M,N,K", [(1, 1000, 4160), (64, 700, 1024), (200, 300, 512)])
def test_masked_matmul_graph_replay(M, N, K):
    """The product captured in a HIP graph (dot products; decode kernel: C
    cleared by a kernel, partial products added atomically; tiled kernel) and replayed
    three times, with C overwritten and other work run eagerly between the
    replays: every replay equals the eagerly launched product."""
    rng = _rng_np(M + 3 * N + 7 * K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    A, B = Digits.empty(M, K), Digits.empty(N, K)
    m.mosaic_mask(to_dev_ring(a), None, None, M, K, out_dig=A)
    m.mosaic_mask(to_dev_ring(b), None, None, N, K, out_dig=B)
    C = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(A, B, M, N, K, C)
    torch.cuda.synchronize()
    eager = to_np_u32(C)
    assert np.array_equal(eager, ring_matmul(a, b.T))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.mosaic_masked_matmul(A, B, M, N, K, C)
    for rep in range(3):
        C.fill_(12345 + rep)
        m.mosaic_mask(to_dev_ring(b), None, None, N, K, out_dig=Digits.empty(N, K))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(to_np_u32(C), eager), rep


@pytest.mark.parametrize("M", [5, 64])
def test_masked_matmul_accumulator_extreme_short_a(M):
    N, K = 40, 32767
    a = np.full((M, K), 0x7F7F7F80, dtype=np.uint32)
    b = np.full((N, K), 0x7F7F7F80, dtype=np.uint32)
    got = _gemm(a, b)
    assert np.all(got == (K * (0x7F7F7F80 ** 2)) % (1 << 32))


@pytest.mark.parametrize("M,N,K", [(70, 50, 40000), (130, 132, 33000), (3, 37, 65600)])
def test_masked_matmul_long_inner_dimension(M, N, K):
    """K >= 2^15 runs as chunks added into C (tiled kernel, epilogues of
    unaligned and aligned rows, and the K-split kernel)."""
    rng = _rng_np(M + N + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    assert np.array_equal(_gemm(a, b), ring_matmul(a, b.T))


@pytest.mark.parametrize("M", [5, 130])
def test_masked_matmul_accumulator_extreme_long_k(M):
    """All digits -128 at K = 70000: one launch would overflow the
    four-product class (4 K 2^14 > 2^31); the chunks keep it exact."""
    N, K = 36, 70000
    a = np.full((M, K), 0x7F7F7F80, dtype=np.uint32)
    b = np.full((N, K), 0x7F7F7F80, dtype=np.uint32)
    got = _gemm(a, b)
    assert np.all(got == (K * (0x7F7F7F80 ** 2)) % (1 << 32))


def test_masked_matmul_accumulator_extreme():
    """All digits -128 (x = 0x7F7F7F80) at the largest supported K: every
    limb product is +2^14, the four-product class reaches 4 K 2^14 < 2^31."""
    M, N, K = 130, 70, 32767
    a = np.full((M, K), 0x7F7F7F80, dtype=np.uint32)
    b = np.full((N, K), 0x7F7F7F80, dtype=np.uint32)
    got = _gemm(a, b)
    ref = (K * (0x7F7F7F80 ** 2)) % (1 << 32)
    assert np.all(got == ref)


@pytest.mark.parametrize("M,K", [(70, 130), (40, 2000)])
def test_masked_matmul_ldc_and_offsets(M, K):
    """Output with a leading dimension > N and operands at a column offset in
    a wider digit buffer; C starts non-zero and only its M x N window may
    change. M = 40 with K = 2000 takes the decode kernel (the window cleared,
    partial products of the workgroups' K ranges added atomically)."""
    rng = _rng_np(11 + M)
    N = 50
    a = _random_ring(rng, (M, K))
    b = _random_ring(rng, (N, K))
    left = Digits.concat(M, [64, K])
    right = Digits.concat(N, [K, 100])
    m.mosaic_mask(to_dev_ring(a), None, None, M, K, out_dig=left[1])
    m.mosaic_mask(to_dev_ring(b), None, None, N, K, out_dig=right[0])
    C = torch.full((M, N + 17), 12345, dtype=torch.int32, device="cuda")
    m.mosaic_masked_matmul(left[1], right[0], M, N, K, C[:, 5:5 + N])
    torch.cuda.synchronize()
    got = to_np_u32(C)
    assert np.array_equal(got[:, 5:5 + N], ring_matmul(a, b.T))
    assert np.all(got[:, :5] == 12345) and np.all(got[:, 5 + N:] == 12345)


def _gemm_words(a_np, b_np, ldb, c0=None, accumulate=False, ldc_extra=0):
    """C (+)= A B^T with A as digits and B as ring words in the first K
    columns of an N x ldb buffer whose other columns hold random words."""
    M, K = a_np.shape
    N = b_np.shape[0]
    A = Digits.empty(M, K)
    m.mosaic_mask(to_dev_ring(a_np), None, None, M, K, out_dig=A)
    wide = _rng_np(ldb + N).integers(0, 2 ** 32, (N, ldb), dtype=np.uint64).astype(np.uint32)
    wide[:, :K] = b_np
    Bw = to_dev_ring(wide)[:, :K]
    C = to_dev_ring(c0 if c0 is not None else np.full((M, N + ldc_extra), 777, dtype=np.uint32))
    m.mosaic_masked_matmul_words(A, Bw, M, N, K, C[:, :N], accumulate=accumulate)
    torch.cuda.synchronize()
    return to_np_u32(C)


@pytest.mark.parametrize("M", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("N,K,ldb", [(33, 64, 64), (100, 576, 580), (300, 1001, 1008), (2049, 1024, 1024),
                                     (37, 1, 4), (130, 4161, 4164)])
def test_masked_matmul_words(M, N, K, ldb):
    """B read as ring words (the integrity check's operand layout): row
    counts of one, two and four 16-row tiles, ragged N and K, a leading
    dimension above K whose extra words are random (A's zero digits past K
    cancel them), and B's last row ending at its K-th word (ldb = K)."""
    rng = _rng_np(M * 3 + N * 5 + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    got = _gemm_words(a, b, ldb, ldc_extra=3)
    assert np.array_equal(got[:, :N], ring_matmul(a, b.T))
    assert np.all(got[:, N:] == 777)


@pytest.mark.parametrize("M,N,K", [(3, 37, 33000), (64, 20, 65600)])
def test_masked_matmul_words_long_k_accumulate(M, N, K):
    """K above one launch's range runs as chunks added into C; with
    accumulate set, C's prior values are kept and the product added."""
    rng = _rng_np(M + N + K)
    a = _random_ring(rng, (M, K), edge=True)
    b = _random_ring(rng, (N, K), edge=True)
    c0 = _random_ring(rng, (M, N))
    got = _gemm_words(a, b, K + (-K) % 4 + 4, c0=c0, accumulate=True)
    assert np.array_equal(got, (c0.astype(np.uint64) + ring_matmul(a, b.T)).astype(np.uint32))
    got = _gemm_words(a, b, K + (-K) % 4, c0=c0, accumulate=False)
    assert np.array_equal(got, ring_matmul(a, b.T))


@pytest.mark.parametrize("M,N,R", [(64, 512, 128), (33, 70, 0), (200, 130, 192), (1, 300, 2560), (8, 33, 64),
                                   (200, 132, 192), (130, 256, 64), (257, 4, 128), (1, 4096, 1536),
                                   (1, 4200, 1536), (16, 4111, 320)])
@pytest.mark.parametrize("with_k", [True, False])
def test_unmask(M, N, R, with_k):
    """Y = Ym - Kc - Q L^T against the oracle; at up to 16 rows the kernel
    takes one 16-column tile per workgroup up to N = 16 x compute units
    (4096 on 256 units) and two above (4111, 4200: ragged last tiles)."""
    rng = _rng_np(M + N + R)
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N)) if with_k else None
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, max(R, 1)), Digits.empty(N, max(R, 1))
    if R:
        m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
        m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    y = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_unmask(to_dev_ring(ym), to_dev_ring(kc) if with_k else None, Q if R else None, L if R else None,
                    M, N, R, y=y)
    torch.cuda.synchronize()
    ref = ym.copy()
    if with_k:
        ref = ring_sub(ref, kc)
    if R:
        ref = ring_sub(ref, ring_matmul(q, l.T))
    assert np.array_equal(y.cpu().numpy(), ref.view(np.int32))


@pytest.mark.parametrize("M", [1, 20, 64])
@pytest.mark.parametrize("case", ["y", "y_and_f32", "f32", "y_is_ym", "y_is_kc", "f32_over_ym", "y_is_ym_and_f32"])
def test_unmask_short_a_outputs(M, case):
    """Unmask with at most 64 rows over several column tiles (N = 700, R =
    1088): for 20 and 64 rows an output that shares no memory with the
    inputs holds the product until the elementwise pass (y, y with y_f32,
    y_f32 alone, and y_f32 when y is in place on ym); in place on ym or kc,
    or y_f32 over ym's memory, and for one row with this small factor, the
    whole-tile kernel runs. Every case equals the oracle."""
    N, R = 700, 1088
    rng = _rng_np(M * 3 + len(case))
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N))
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, R), Digits.empty(N, R)
    m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
    m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    ymd, kcd = to_dev_ring(ym), to_dev_ring(kc)
    sr = torch.rand(M, device="cuda") * 1e-3
    sc = torch.rand(N, device="cuda") * 1e-3
    want_f32 = case in ("y_and_f32", "f32", "f32_over_ym", "y_is_ym_and_f32")
    y = {"y": torch.empty((M, N), dtype=torch.int32, device="cuda"),
         "y_and_f32": torch.empty((M, N), dtype=torch.int32, device="cuda"),
         "y_is_ym": ymd, "y_is_kc": kcd, "y_is_ym_and_f32": ymd}.get(case)
    yf = None
    if case in ("y_and_f32", "f32", "y_is_ym_and_f32"):
        yf = torch.empty((M, N), dtype=torch.float32, device="cuda")
    elif case == "f32_over_ym":
        yf = ymd.view(torch.float32)
    bd, bn = _bias(N, "aligned" if case in ("f32", "f32_over_ym") else None, M + 11)
    m.mosaic_unmask(ymd, kcd, Q, L, M, N, R, y=y, s_rows=sr if want_f32 else None,
                    s_cols=sc if want_f32 else None, y_f32=yf, bias=bd)
    torch.cuda.synchronize()
    yi = ring_sub(ring_sub(ym, kc), ring_matmul(q, l.T)).view(np.int32)
    if y is not None:
        assert np.array_equal(y.cpu().numpy(), yi)
    if want_f32:
        ref = (yi.astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
        if bd is not None:
            ref = (ref + bn).astype(np.float32)
        assert np.array_equal(yf.cpu().numpy(), ref)


@pytest.mark.parametrize("with_f32", [False, True])
def test_unmask_one_row_large_factor(with_f32):
    """One row against a large factor (N = 16384, R = 2048: 128 MiB of
    digits): the product goes through the disjoint output and the
    elementwise pass; equal to the oracle."""
    M, N, R = 1, 16384, 2048
    rng = _rng_np(77 + with_f32)
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N))
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, R), Digits.empty(N, R)
    m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
    m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    y = torch.empty((M, N), dtype=torch.int32, device="cuda")
    sr = torch.rand(M, device="cuda") * 1e-3
    sc = torch.rand(N, device="cuda") * 1e-3
    yf = torch.empty((M, N), dtype=torch.float32, device="cuda") if with_f32 else None
    bd, bn = _bias(N, "offset" if with_f32 else None, 99)
    m.mosaic_unmask(to_dev_ring(ym), to_dev_ring(kc), Q, L, M, N, R, y=y, s_rows=sr if with_f32 else None,
                    s_cols=sc if with_f32 else None, y_f32=yf, bias=bd)
    torch.cuda.synchronize()
    yi = ring_sub(ring_sub(ym, kc), ring_matmul(q, l.T)).view(np.int32)
    assert np.array_equal(y.cpu().numpy(), yi)
    if with_f32:
        ref = (yi.astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
        ref = (ref + bn).astype(np.float32)
        assert np.array_equal(yf.cpu().numpy(), ref)


def _words_window(rng, q, layout):
    """q (M x R ring words) on the device as a 16-byte aligned view with
    rows a multiple of 4 words apart: its own rows padded to 4 words
    ("tight") or a column window of a wider matrix ("wide", like the Q
    columns of [Y' | Q]). The words around the view are random."""
    M, R = q.shape
    R4 = 4 * ((R + 3) // 4)
    width, c0 = (R4, 0) if layout == "tight" else (R4 + 16, 4)
    big = _random_ring(rng, (M, width))
    big[:, c0: c0 + R] = q
    return to_dev_ring(big)[:, c0: c0 + R]


@pytest.mark.parametrize("M,N,R", [(1, 300, 2560), (8, 33, 64), (1, 4096, 1536), (1, 4200, 1536),
                                   (16, 4111, 320), (3, 700, 1088), (1, 70, 5), (2, 130, 67), (5, 64, 0),
                                   (1, 16384, 2048)])
@pytest.mark.parametrize("layout", ["tight", "wide"])
def test_unmask_words(M, N, R, layout):
    """Q given as ring words (at most 16 rows): Y = Ym - Kc - Q L^T equals
    the oracle, for ragged R (the words after column R in a row are other
    data; L's zero digit padding cancels them), ragged column tiles of N and
    a 128 MiB factor (16384 x 2048)."""
    rng = _rng_np(7 * M + N + R + len(layout))
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N))
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    L = Digits.empty(N, max(R, 1))
    if R:
        m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    y = torch.empty((M, N), dtype=torch.int32, device="cuda")
    m.mosaic_unmask_words(to_dev_ring(ym), to_dev_ring(kc), _words_window(rng, q, layout) if R else None,
                          L if R else None, M, N, R, y=y)
    torch.cuda.synchronize()
    ref = ring_sub(ym, kc)
    if R:
        ref = ring_sub(ref, ring_matmul(q, l.T))
    assert np.array_equal(y.cpu().numpy(), ref.view(np.int32))


@pytest.mark.parametrize("M", [1, 16])
@pytest.mark.parametrize("case", ["y_and_f32_bias", "f32", "y_is_ym", "y_is_kc", "y_no_kc"])
def test_unmask_words_outputs(M, case):
    """The word form's outputs: y with the dequantised y_f32 and a bias,
    y_f32 alone, y in place on ym or on kc, and y without K_c; bit-identical
    to mosaic_unmask with the digits of the same Q and to the oracle."""
    N, R = 700, 1088
    rng = _rng_np(M * 5 + len(case))
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N)) if case != "y_no_kc" else np.zeros((M, N), dtype=np.uint32)
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, R), Digits.empty(N, R)
    m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
    m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    sr = torch.rand(M, device="cuda") * 1e-3
    sc = torch.rand(N, device="cuda") * 1e-3
    want_f32 = case in ("y_and_f32_bias", "f32")
    bd, bn = _bias(N, "aligned" if case == "y_and_f32_bias" else None, M + 3)
    outs = []
    for words in (True, False):
        ymd, kcd = to_dev_ring(ym), (to_dev_ring(kc) if case != "y_no_kc" else None)
        y = {"y_and_f32_bias": torch.empty((M, N), dtype=torch.int32, device="cuda"),
             "y_no_kc": torch.empty((M, N), dtype=torch.int32, device="cuda"),
             "y_is_ym": ymd, "y_is_kc": kcd}.get(case)
        yf = torch.empty((M, N), dtype=torch.float32, device="cuda") if want_f32 else None
        kw = dict(y=y, s_rows=sr if want_f32 else None, s_cols=sc if want_f32 else None, y_f32=yf, bias=bd)
        if words:
            m.mosaic_unmask_words(ymd, kcd, _words_window(rng, q, "wide"), L, M, N, R, **kw)
        else:
            m.mosaic_unmask(ymd, kcd, Q, L, M, N, R, **kw)
        torch.cuda.synchronize()
        outs.append((y.cpu().numpy() if y is not None else None, yf.cpu().numpy() if yf is not None else None))
    yi = ring_sub(ring_sub(ym, kc), ring_matmul(q, l.T)).view(np.int32)
    (yw, fw), (yd, fd) = outs
    if yw is not None:
        assert np.array_equal(yw, yi) and np.array_equal(yd, yi)
    if want_f32:
        ref = (yi.astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
        if bd is not None:
            ref = (ref + bn).astype(np.float32)
        assert np.array_equal(fw, ref) and np.array_equal(fd, ref)


@pytest.mark.parametrize("M", [130, 257])
@pytest.mark.parametrize("target", ["ym", "kc"])
def test_unmask_in_place_tiled(M, target):
    """Unmask through the tiled kernel (more than 64 rows) with y in place on
    ym or on kc: each thread loads its chunks' inputs before storing."""
    N, R = 300, 192
    rng = _rng_np(M + 11 * len(target))
    ym = _random_ring(rng, (M, N))
    kc = _random_ring(rng, (M, N))
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, R), Digits.empty(N, R)
    m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
    m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    ymd, kcd = to_dev_ring(ym), to_dev_ring(kc)
    y = ymd if target == "ym" else kcd
    m.mosaic_unmask(ymd, kcd, Q, L, M, N, R, y=y)
    torch.cuda.synchronize()
    ref = ring_sub(ring_sub(ym, kc), ring_matmul(q, l.T)).view(np.int32)
    assert np.array_equal(y.cpu().numpy(), ref)


def _bias(N, kind, seed):
    """None, a 16-byte aligned bias, or one at a 4-byte offset (the tiled
    kernel then takes its epilogue of unaligned rows)."""
    if kind is None:
        return None, 0.0
    b = torch.from_numpy(_rng_np(seed).standard_normal(N + 1).astype(np.float32)).cuda()
    b = b[:N] if kind == "aligned" else b[1:]
    return b, b.cpu().numpy()[None, :]


@pytest.mark.parametrize("M,N", [(40, 90), (150, 90), (150, 92), (300, 260)])
@pytest.mark.parametrize("bias", [None, "aligned", "offset"])
def test_unmask_dequantised(M, N, bias):
    """y_f32 = (y s_rows) s_cols (+ bias), each step rounded to fp32, equal
    bit for bit to the same steps in numpy."""
    rng = _rng_np(5 + M + N)
    R = 64
    ym = _random_ring(rng, (M, N))
    q = _random_ring(rng, (M, R))
    l = _random_ring(rng, (N, R))
    Q, L = Digits.empty(M, R), Digits.empty(N, R)
    m.mosaic_mask(to_dev_ring(q), None, None, M, R, out_dig=Q)
    m.mosaic_mask(to_dev_ring(l), None, None, N, R, out_dig=L)
    sr = torch.rand(M, device="cuda") * 1e-3
    sc = torch.rand(N, device="cuda") * 1e-3
    yf = torch.empty((M, N), dtype=torch.float32, device="cuda")
    bd, bn = _bias(N, bias, M * N)
    m.mosaic_unmask(to_dev_ring(ym), None, Q, L, M, N, R, s_rows=sr, s_cols=sc, y_f32=yf, bias=bd)
    torch.cuda.synchronize()
    yi = ring_sub(ym, ring_matmul(q, l.T)).view(np.int32)
    ref = (yi.astype(np.float32) * sr.cpu().numpy()[:, None]) * sc.cpu().numpy()[None, :]
    if bd is not None:
        ref = (ref + bn).astype(np.float32)
    assert np.array_equal(yf.cpu().numpy(), ref)


@pytest.mark.parametrize("rows,n,block", [(3, 16, 16), (4, 32, 32), (5, 64, 64), (3, 128, 128), (2, 4096, 256),
                                          (3, 512, 512), (4, 1024, 1024), (3, 2048, 2048), (3, 28672, 4096),
                                          (6, 8192, 8192), (3, 24576, 8192), (2, 16384, 16384),
                                          (2, 32768, 32768)])
@pytest.mark.parametrize("inverse", [False, True])
def test_hadamard(rows, n, block, inverse):
    x = _rng_np(n + rows).standard_normal((rows, n)).astype(np.float32)
    x[0, 3] *= 50.0
    signs = smp.sample_signs(n, SEED, 1)
    xd = torch.from_numpy(x).cuda()
    y = torch.empty_like(xd)
    m.mosaic_hadamard_rotate(xd, y, block=block, signs=torch.from_numpy(signs).cuda(), inverse=inverse)
    torch.cuda.synchronize()
    ref = ohad.rotate(x.astype(np.float64), signs, block=block, inverse=inverse)
    err = np.max(np.abs(y.cpu().numpy().astype(np.float64) - ref), axis=1) / np.max(np.abs(ref), axis=1)
    assert np.all(err <= 1e-5), err.max()


@pytest.mark.parametrize("rows,b", [(3, 256), (2, 512), (5, 1024)])
@pytest.mark.parametrize("inverse", [False, True])
def test_hadamard28(rows, b, inverse):
    """H_28 (x) H_b rotation (n = 28 b) against the oracle's float64
    rotation: max relative error per row <= 1e-5."""
    n = 28 * b
    x = _rng_np(n + rows).standard_normal((rows, n)).astype(np.float32)
    x[0, 5] *= 50.0
    signs = smp.sample_signs(n, SEED, 2)
    xd = torch.from_numpy(x).cuda()
    y = torch.empty_like(xd)
    m.mosaic_hadamard28_rotate(xd, y, signs=torch.from_numpy(signs).cuda(), inverse=inverse)
    torch.cuda.synchronize()
    ref = ohad.rotate_kron28(x.astype(np.float64), signs, inverse=inverse)
    err = np.max(np.abs(y.cpu().numpy().astype(np.float64) - ref), axis=1) / np.max(np.abs(ref), axis=1)
    assert np.all(err <= 1e-5), err.max()


def test_hadamard28_in_place_roundtrip_and_no_signs():
    rows, n = 4, 28672
    x = _rng_np(28).standard_normal((rows, n)).astype(np.float32)
    signs = torch.from_numpy(smp.sample_signs(n, SEED, 3)).cuda()
    xd = torch.from_numpy(x).cuda()
    m.mosaic_hadamard28_rotate(xd, xd, signs=signs)
    m.mosaic_hadamard28_rotate(xd, xd, signs=signs, inverse=True)
    torch.cuda.synchronize()
    back = xd.cpu().numpy()
    assert np.max(np.abs(back - x) / np.max(np.abs(x), axis=1, keepdims=True)) <= 1e-5
    y = torch.empty((rows, n), dtype=torch.float32, device="cuda")
    m.mosaic_hadamard28_rotate(torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    ref = ohad.rotate_kron28(x.astype(np.float64), np.ones(n, dtype=np.int8))
    assert np.max(np.abs(y.cpu().numpy() - ref) / np.max(np.abs(ref), axis=1, keepdims=True)) <= 1e-5


def test_hadamard_in_place_roundtrip_and_no_signs():
    rows, n = 8, 8192
    x = _rng_np(9).standard_normal((rows, n)).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    signs = torch.from_numpy(smp.sample_signs(n, SEED, 2)).cuda()
    m.mosaic_hadamard_rotate(xd, xd, signs=signs)
    m.mosaic_hadamard_rotate(xd, xd, signs=signs, inverse=True)
    torch.cuda.synchronize()
    back = xd.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(back - x) / np.max(np.abs(x), axis=1, keepdims=True)) <= 1e-5
    y = torch.empty((rows, n), dtype=torch.float32, device="cuda")
    m.mosaic_hadamard_rotate(torch.from_numpy(x).cuda(), y)
    torch.cuda.synchronize()
    ref = ohad.rotate(x.astype(np.float64), np.ones(n, dtype=np.int8))
    assert np.max(np.abs(y.cpu().numpy() - ref) / np.max(np.abs(ref), axis=1, keepdims=True)) <= 1e-5


@pytest.mark.parametrize("rows,n,qmax", [(5, 100, 127), (16, 8192, 1997), (3, 28672, 567), (2, 64, 1),
                                         (7, 102, 127), (4, 4100, 300), (3, 1024, 127), (3, 2000, 127),
                                         (2, 4096, 255), (2, 9000, 127), (2, 16384, 1000), (2, 16388, 77),
                                         (2, 40000, 127), (2, 65536, 300), (2, 70000, 511)])
@pytest.mark.parametrize("offset", [0, 1])
def test_quantize(rows, n, qmax, offset):
    """offset 1 reads rows that start one float into a wider buffer (not
    16-byte aligned): the general kernel; offset 0 with n % 4 == 0: the
    register-resident kernel (256 threads up to n = 16384, 1024 threads up
    to 65536; each size class also with a ragged row) or, beyond, the
    two-pass vector kernel."""
    x = _rng_np(n).standard_normal((rows, n)).astype(np.float32)
    x[1] = 0.0
    wide = torch.zeros((rows, n + 4), dtype=torch.float32, device="cuda")
    wide[:, offset: offset + n] = torch.from_numpy(x).cuda()
    xd = wide[:, offset: offset + n]
    q = torch.empty((rows, n), dtype=torch.int32, device="cuda")
    dig = Digits.empty(rows, n)
    dig.buf.fill_(0x55)
    sc = torch.empty(rows, dtype=torch.float32, device="cuda")
    m.mosaic_quantize_rows(xd, qmax, q=q, q_dig=dig, scale=sc)
    torch.cuda.synchronize()
    qr, sr = oquant.quantize_rows(x, qmax)
    assert np.array_equal(sc.cpu().numpy(), sr)
    assert np.array_equal(q.cpu().numpy(), qr)
    assert np.array_equal(unpack_digits(dig), qr.view(np.uint32))
    assert pad_is_zero(dig)


def test_quantize_single_outputs():
    """Codes only and digits only; a call with neither is rejected."""
    rows, n, qmax = 6, 1024, 511
    x = _rng_np(99).standard_normal((rows, n)).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    qr, sr = oquant.quantize_rows(x, qmax)
    q = torch.empty((rows, n), dtype=torch.int32, device="cuda")
    m.mosaic_quantize_rows(xd, qmax, q=q)
    dig = Digits.empty(rows, n)
    m.mosaic_quantize_rows(xd, qmax, q_dig=dig)
    sc = torch.empty(rows, dtype=torch.float32, device="cuda")
    with pytest.raises(m.MosaicError):
        m.mosaic_quantize_rows(xd, qmax, scale=sc)
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), qr)
    assert np.array_equal(unpack_digits(dig), qr.view(np.uint32))
