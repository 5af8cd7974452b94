"""The dispatch rules at the sizes where they change, and over the launch
limits (no GPU needed)."""
import pytest

from tests.dispatch_util import mask_route

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
