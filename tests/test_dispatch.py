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


@pytest.mark.parametrize("D,ordered", [(3, True), (4, False)])
def test_sums_do_not_order_points_that_no_order_can_help(D, ordered):
    """From 10^10 pairs on sums may order their points (16 bytes a point).  At these sizes the rule
    asks for a range of about 270 log2 units at D = 3 and of 700 at D = 4, where the matrix-core path's box
    spans at most 4 * 128, times (32 / 31)^2 for the bulk's."""
    cols = 90_001
    rows = 10 ** 10 // cols
    below, above = (kred.scratch_bytes("gauss", "sum", m, cols, D, 1, sigma=0.1) for m in (rows, rows + 1))
    assert (above - below >= 16 * (rows + cols)) == ordered
