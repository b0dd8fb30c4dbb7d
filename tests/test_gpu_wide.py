"""GPU vs oracle for the 32x32-tile sums at D <= 16 and products at D <= 4.

Sums with 5 <= D <= 16 (one to four signal columns on the vector ALU, up to 16
per call on the matrix cores) or with more than four signal columns, and the
vector-Jacobian product with any cotangent width.  Sizes straddle the 32-row
and 32-column blocks, the 128-column tiles and the 256 rows of a workgroup;
D every chunk count of the K slots; E every operand form and slice edge.
Tolerance of a row, a bound: the exponent t = c d of a term is rounded in at
most 15 groups, each below 2^-24 t, so the term is off by less than ln 2 times
15 2^-24 t < 11 2^-24 t of itself; the rest (products, the fp32 sum) is ten times
the 2^-24 sqrt(N) growth of an fp32 sum of its terms.  Beyond the box limit the
direct form must run.
"""
import numpy as np
import pytest

import oracle
from helpers import SUM_TOL, dev, host, norm_err
from paper_2004_11127_amd import kred

pytestmark = pytest.mark.gpu
FAST = kred.FLAG_FAST | kred.FLAG_PROFILE


@pytest.fixture(scope="module")
def ctx():
    with kred.Context(0) as c:
        yield c


def _allow(k, d2, sigma, size, N):
    """The tolerance of sum_j k_ij s_ij with |s_ij| = size[i, j, ...] (see above)."""
    t = d2 * (1.4426950408889634 / (2 * sigma * sigma))
    w = 10 * np.sqrt(N) + 11 * t
    return 2.0 ** -24 * np.einsum("ij,ij...->i...", k * w, size) + 1e-30


def _pairs(x, y, sigma):
    d2 = ((x[:, None].astype(np.float64) - y[None]) ** 2).sum(-1)
    return np.exp(-d2 / (2 * sigma * sigma)), d2


SIZES = [(1, 1), (31, 33), (257, 128), (256, 129), (300, 1000), (65, 3001)]


@pytest.mark.parametrize("M,N", SIZES)
@pytest.mark.parametrize("D,E", [(5, 1), (6, 1), (7, 2), (8, 4), (9, 5), (10, 1), (11, 16), (12, 3), (13, 17),
                                 (14, 1), (15, 4), (16, 1), (16, 33), (1, 5), (2, 16), (3, 20), (4, 64)])
@pytest.mark.parametrize("C", [0, 3])
def test_sums(ctx, M, N, D, E, C):
    rng = np.random.default_rng(D * 100 + E)
    x = (5 + rng.standard_normal((M, D))).astype(np.float32)     # off the origin
    y = (5 + rng.standard_normal((N, D))).astype(np.float32)
    b = rng.standard_normal((N, E)).astype(np.float32)
    sigma = 0.7 * np.sqrt(D)
    ctx.profile_collect()
    got = host(ctx.run("gauss", "sum", dev(x), dev(y), dev(b), sigma=sigma, col_blocks=C, flags=FAST))
    assert ctx.profile_collect()[2] == "wide_kernel"
    ref, norm = oracle.kernel_sum("gauss", x, y, b, sigma=sigma)
    k, d2 = _pairs(x, y, sigma)
    assert np.all(np.abs(got - ref) <= _allow(k, d2, sigma, np.broadcast_to(np.abs(b)[None], (M, N, E)), N))


@pytest.mark.parametrize("M,N", SIZES)
@pytest.mark.parametrize("D,E", [(1, 2), (2, 5), (3, 3), (3, 6), (3, 10), (3, 11), (3, 16), (3, 17), (3, 40), (4, 1),
                                 (4, 16)])
@pytest.mark.parametrize("C", [0, 3])
def test_products(ctx, M, N, D, E, C):
    rng = np.random.default_rng(D * 100 + E)
    x = rng.uniform(4, 5, (M, D)).astype(np.float32)
    y = rng.uniform(4, 5, (N, D)).astype(np.float32)
    b = rng.standard_normal((N, E)).astype(np.float32)
    e = rng.standard_normal((M, E)).astype(np.float32)
    sigma = 0.3
    ctx.profile_collect()
    gx, gy, gb = ctx.gauss_backward(dev(x), dev(y), dev(b), dev(e), sigma=sigma, col_blocks=C,
                                    gb=E > 4, flags=FAST)
    assert ctx.profile_collect()[2] == "wide_kernel"
    ref, norm = oracle.gauss_vjp(x, y, b, e, sigma)
    # <e, b> cancels: its own rounding scales with sum |e b|
    k, d2 = _pairs(x, y, sigma)
    size = (np.abs(e) @ np.abs(b).T)[:, :, None] * np.abs(y[None].astype(np.float64) - x[:, None]) / sigma ** 2
    assert np.all(np.abs(host(gx) - ref) <= _allow(k, d2, sigma, size, N))
    ref, _ = oracle.gauss_vjp(y, x, e, b, sigma)
    assert np.all(np.abs(host(gy) - ref) <= _allow(k.T, d2.T, sigma, size.transpose(1, 0, 2), M))
    if E > 4:
        ref, norm = oracle.kernel_sum("gauss", y, x, e, sigma=sigma)
        size = np.broadcast_to(np.abs(e)[None], (N, M, E))
        assert np.all(np.abs(host(gb) - ref) <= _allow(k.T, d2.T, sigma, size, M))


@pytest.mark.parametrize("D,E", [(10, 1), (16, 4), (7, 16), (3, 16)])
def test_near_and_beyond_the_box_limit(ctx, D, E):
    rng = np.random.default_rng(D)
    x = rng.uniform(0, 1, (200, D)).astype(np.float32)
    y = rng.uniform(0, 1, (700, D)).astype(np.float32)
    x[0], y[0] = 0, 1                  # the whole unit box: R^2 = D / 4
    b = rng.standard_normal((700, E)).astype(np.float32)
    limit = 2048.0 if D <= 3 else 256.0
    for L, kernel in ((0.97 * limit, "wide_kernel"), (1.03 * limit, "sum_kernel")):
        sigma = float(np.sqrt(1.4426950408889634 * D / 4 / L / 2))
        ctx.profile_collect()
        got = host(ctx.run("gauss", "sum", dev(x), dev(y), dev(b), sigma=sigma, flags=FAST))
        assert ctx.profile_collect()[2] == kernel
        ref, norm = oracle.kernel_sum("gauss", x, y, b, sigma=sigma)
        assert norm_err(got, ref, norm) <= SUM_TOL


def test_products_beyond_the_box_limit(ctx):
    rng = np.random.default_rng(1)
    x = rng.uniform(0, 1, (200, 3)).astype(np.float32)
    y = np.concatenate([x[:100] + np.float32(0.002), rng.uniform(0, 1, (600, 3)).astype(np.float32)])
    b, e = (rng.standard_normal((n, 8)).astype(np.float32) for n in (700, 200))
    ctx.profile_collect()
    gx = ctx.gauss_backward(dev(x), dev(y), dev(b), dev(e), sigma=0.005, gy=False, gb=False, flags=FAST)[0]
    assert ctx.profile_collect()[2] == "vjp_kernel"
    ref, norm = oracle.gauss_vjp(x, y, b, e, 0.005)
    assert norm_err(host(gx), ref, norm) <= SUM_TOL


def _ratio(got, direct, ref):
    """2-norm of the error against the direct form's."""
    return np.linalg.norm(got - ref) / np.linalg.norm(direct - ref)


# An error that is alike for all columns of a row does not average out as the
# rounding of a long sum does, so the columns are many.  Both forms round every
# term by a few 2^-24; 1.25 allows for the spread of two such errors over the rows.
@pytest.mark.parametrize("D,E,sigma,kernel", [
    (3, 3, 0.1, "wide_kernel"), (3, 16, 0.2, "wide_kernel"), (2, 3, 0.3, "wide_kernel"), (4, 8, 0.3, "wide_kernel"),
    (2, 8, 0.1, "wide_kernel"), (3, 6, 0.05, "vjp_kernel"), (1, 6, 0.05, "vjp_kernel"),
])
@pytest.mark.parametrize("positive", [False, True])
def test_products_are_as_exact_as_the_direct_form(ctx, D, E, sigma, kernel, positive):
    rng = np.random.default_rng(D * 10 + E)
    M, N = 2300, 120011                      # 2^28 pairs: the default takes the wide kernel
    x = rng.uniform(0, 1, (M, D)).astype(np.float32)
    y = rng.uniform(0, 1, (N, D)).astype(np.float32)
    w = (lambda n: rng.uniform(0, 1, (n, E))) if positive else (lambda n: rng.standard_normal((n, E)))
    b, e = w(N).astype(np.float32), w(M).astype(np.float32)
    rows = np.arange(0, M, 9)
    ref, _ = oracle.gauss_vjp(x, y, b, e, float(np.float32(sigma)), rows=rows)
    dx, dy, db, de = dev(x), dev(y), dev(b), dev(e)
    out = {}
    for flags in (0, kred.FLAG_DIRECT):
        ctx.profile_collect()
        out[flags] = host(ctx.gauss_backward(dx, dy, db, de, sigma=sigma, gy=False, gb=False,
                                             flags=flags | kred.FLAG_PROFILE)[0])[rows]
        assert ctx.profile_collect()[2] == ("vjp_kernel" if flags else kernel)
    assert _ratio(out[0], out[kred.FLAG_DIRECT], ref) <= 1.25


@pytest.mark.parametrize("D,sigma", [(3, 0.1), (2, 0.1), (4, 0.2), (3, 0.02), (7, 0.6)])
@pytest.mark.parametrize("positive", [False, True])
def test_sums_are_as_exact_as_the_direct_form(ctx, D, sigma, positive):
    rng = np.random.default_rng(D)
    M, N, E = 600, 500009, 16
    x = rng.uniform(0, 1, (M, D)).astype(np.float32)
    y = rng.uniform(0, 1, (N, D)).astype(np.float32)
    b = (rng.uniform(0, 1, (N, E)) if positive else rng.standard_normal((N, E))).astype(np.float32)
    rows = np.arange(0, M, 6)
    ref, _ = oracle.kernel_sum("gauss", x, y, b, sigma=float(np.float32(sigma)), rows=rows)
    out = {}
    for flags in (0, kred.FLAG_DIRECT):
        out[flags] = host(ctx.run("gauss", "sum", dev(x), dev(y), dev(b), sigma=sigma, flags=flags))[rows]
    assert _ratio(out[0], out[kred.FLAG_DIRECT], ref) <= 1.25


@pytest.mark.parametrize("low", [-3.4028235e38, 3.4028235e38])
def test_weights_of_the_types_largest_values(ctx, low):
    """A head of three bf16 parts rounded to nearest would be infinite there."""
    rng = np.random.default_rng(2)
    x, y = rng.uniform(0, 1, (70, 3)).astype(np.float32), rng.uniform(0, 1, (300, 3)).astype(np.float32)
    b = rng.standard_normal((300, 8)).astype(np.float32)
    b[5, 3] = low
    got = host(ctx.run("gauss", "sum", dev(x), dev(y), dev(b), sigma=0.4, flags=FAST))
    ref, norm = oracle.kernel_sum("gauss", x, y, b, sigma=float(np.float32(0.4)))
    assert norm_err(got, ref, norm) <= SUM_TOL
    e = (rng.standard_normal((70, 8)) * 1e-3).astype(np.float32)
    gx = host(ctx.gauss_backward(dev(x), dev(y), dev(b), dev(e), sigma=0.4, gy=False, gb=False, flags=FAST)[0])
    ref, norm = oracle.gauss_vjp(x, y, b, e, float(np.float32(0.4)))
    assert norm_err(gx, ref, norm) <= SUM_TOL
