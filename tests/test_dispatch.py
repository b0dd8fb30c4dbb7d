"""Which kernel a call is sent to, where that depends on its sizes alone (CPU: by the scratch it asks for)."""
import pytest

from paper_2004_11127_amd import kred


@pytest.mark.parametrize("K,reduction", [(1, "argkmin"), (10, "argkmin"), (64, "kmin"), (0, "min")])
def test_lists_of_more_rows_than_a_launch_holds(K, reduction):
    """The ordered lists take a wave for every four rows, so 2^28 rows would need 2^32 threads; the
    order is 16 bytes a point."""
    rows, cols = 1 << 28, 100_000
    below = kred.scratch_bytes("sqdist", reduction, rows - 1, cols, 3, 0, K=K)
    assert below >= 16 * (rows - 1 + cols)
    assert kred.scratch_bytes("sqdist", reduction, rows, cols, 3, 0, K=K) < 4 * rows


def test_sums_of_more_items_than_a_launch_holds():
    """The 32x32-tile sums take a thread for every row and column block."""
    kw = dict(sigma=1.0, col_blocks=256)
    for rows, wide in (((1 << 24) - 1, True), (1 << 24, False)):
        got = kred.scratch_bytes("gauss", "sum", rows, 1 << 20, 10, 1, **kw)
        direct = kred.scratch_bytes("gauss", "sum", rows, 1 << 20, 10, 1, flags=kred.FLAG_DIRECT, **kw)
        assert (got > direct) == wide and (wide or got == direct)
