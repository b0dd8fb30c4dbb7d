"""GPU vs oracle for the spatially ordered paths (D <= 4).

Both clouds are sorted along a Hilbert curve, and boxes of 64 columns (and of
64 such subtiles) decide which columns a row visits.  The neighbour lists must
equal the oracle's bit for bit on integer coordinates, ties by the lowest
index, whatever order the columns come in; the sums leave out only what lies
below 2^-30 of a row's normaliser, so they keep the parity bar and agree with
the call in place (a column split given by the caller) to fp32 rounding.
Sizes straddle a subtile, 64 subtiles and 64 x 64 subtiles, the row counts per
wave, and the rules' limits.
"""
import numpy as np
import pytest

import oracle
from helpers import LSE_TOL, SUM_TOL, dev, fast_limit, host, lse_err, norm_err
from paper_2004_11127_amd import kred

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    with kred.Context(0) as c:
        yield c


def _rows(rng, M, n=96):
    return np.sort(rng.choice(M, min(M, n), replace=False)).astype(np.int64)


def _lists(ctx, x, y, K, reduction="argkmin"):
    ctx.profile_collect()
    out = host(ctx.run("sqdist", reduction, dev(x), dev(y), K=K, flags=kred.FLAG_PROFILE))
    assert ctx.profile_collect()[2] == "near_kernel"
    return out


# M, N, D, K, coordinates 0 .. top
LATTICE = [
    (4096, 4096, 3, 10, 15), (4097, 4161, 3, 2, 15), (32771, 513, 3, 16, 9), (513, 40000, 3, 5, 40),
    (16384, 16384, 3, 1, 30), (16385, 16449, 2, 1, 200), (1100, 4095, 3, 64, 7), (70001, 4160, 2, 10, 64),
    (5000, 262145 + 4096, 3, 10, 60), (20001, 20000, 1, 4, 5000), (9001, 9002, 4, 12, 9), (600, 300001, 4, 33, 12),
]


@pytest.mark.parametrize("M,N,D,K,top", LATTICE)
def test_lists_on_a_lattice(ctx, M, N, D, K, top):
    rng = np.random.default_rng(M + N)
    x = rng.integers(0, top + 1, (M, D)).astype(np.float32)
    y = rng.integers(0, top + 1, (N, D)).astype(np.float32)      # many equal points and distances
    rows = _rows(rng, M)
    got = _lists(ctx, x, y, K)
    want, d = oracle.argkmin(x, y, K, rows=rows)
    assert np.array_equal(got[rows], want)
    assert np.array_equal(_lists(ctx, x, y, K, "kmin")[rows], d.astype(np.float32))


@pytest.mark.parametrize("K", [2, 10])
@pytest.mark.parametrize("case", ["one point", "far clouds", "outliers", "line", "wide"])
def test_lists_on_awkward_clouds(ctx, case, K):
    rng = np.random.default_rng(K)
    M, N = 5001, 6001
    x = rng.integers(0, 40, (M, 3)).astype(np.float32)
    y = rng.integers(0, 40, (N, 3)).astype(np.float32)
    if case == "one point":
        y[:] = y[0]
    elif case == "far clouds":
        x += np.float32(1000)
    elif case == "outliers":
        x[::50] *= 60
        y[::70] *= 55
    elif case == "line":
        x[:, 1:] = 3
        y[:, 1:] = 3
    else:
        x *= 40        # R^2 far beyond the matrix-core ranking's limit
        y *= 40
    rows = _rows(rng, M)
    assert np.array_equal(_lists(ctx, x, y, K)[rows], oracle.argkmin(x, y, K, rows=rows)[0])


def test_lists_of_real_points(ctx):
    """Not exact distances: each list's distances are the K smallest to fp32 rounding."""
    rng = np.random.default_rng(3)
    c = rng.uniform(0, 1, (8, 3))
    x = (c[rng.integers(0, 8, 70003)] + 0.05 * rng.standard_normal((70003, 3))).astype(np.float32)
    y = (c[rng.integers(0, 8, 90001)] + 0.05 * rng.standard_normal((90001, 3))).astype(np.float32)
    rows = _rows(rng, 70003, 256)
    got = _lists(ctx, x, y, 10)[rows]
    _, d = oracle.argkmin(x, y, 10, rows=rows)
    mine = ((x[rows, None].astype(np.float64) - y[got].astype(np.float64)) ** 2).sum(-1)
    # the direct form's rounding: D + 1 operations on each side of a comparison
    assert np.all(np.abs(mine - d) <= 8 * 2.0 ** -24 * d)
    near, j = _lists(ctx, x, y, 1, "min"), _lists(ctx, x, y, 1, "argmin")
    assert np.all(np.abs(near[rows, 0] - d[:, 0]) <= 4 * 2.0 ** -24 * d[:, 0])
    assert np.array_equal(j[rows, 0], got[:, 0])


def _clouds(rng, M, N, D, data):
    if data == "mixture":
        c = rng.uniform(0, 1, (8, D))
        f = lambda n: c[rng.integers(0, 8, n)] + 0.05 * rng.standard_normal((n, D))
        x, y = f(M), f(N)
    else:
        x, y = rng.uniform(0, 1, (M, D)), rng.uniform(0, 1, (N, D))
    return x.astype(np.float32), y.astype(np.float32)


def _bulk(x, y, d):
    """The span of 31 / 32 of the device's sample along d, scaled to the whole: 128 points of each cloud, one
    from a pseudo-random place in each 128th."""
    v = []
    for p in (x, y):
        for u in range(128):
            t, n = u + (128 if p is y else 0), len(p)
            at, end = n * u // 128, n * (u + 1) // 128
            v.append(p[min(at + (((t + 1) * 2654435761 & 0xFFFFFFFF) >> 8) % max(end - at, 1), n - 1), d])
    q = np.sort(np.array(v))[4::8]
    return float(q[31] - q[0]) * 32 / 31


def _ordered(x, y, c):
    """Whether a sum with exponent -c |x - y|^2 (log2 units) takes the ordered kernel: the matrix-core path's box
    limit holds, and the clouds' bulk spans more than the rule asks at these sizes."""
    (M, D), N = x.shape, len(y)
    half = (np.maximum(x.max(0), y.max(0)) - np.minimum(x.min(0), y.min(0))) / 2
    f = (256 / M) ** (1 / D) + (64 / N) ** (1 / D)
    return (M * N >= 1e10 and f < 0.63 and c * (half ** 2).sum() <= fast_limit(D, False)
            and c * sum(_bulk(x, y, d) ** 2 for d in range(D)) >= 45 / (0.63 - f) ** 2)


def test_far_points_do_not_make_an_order_useful():
    rng = np.random.default_rng(1)
    x, y = rng.uniform(0, 1, (2, 100000, 3)).astype(np.float32)
    c = 1.4426950408889634 / (2 * 0.2 ** 2)
    assert not _ordered(x, y, c) and _ordered(x, y, 16 * c)
    x[5] = 6
    assert not _ordered(x, y, c)


@pytest.mark.parametrize("formula,E", [("gauss", 1), ("gauss", 3), ("gauss_gradx", 1), ("sinkhorn", 1)])
@pytest.mark.parametrize("M,N,D,data,sigma", [
    (100001, 100130, 3, "mixture", 0.05), (100000, 100064, 2, "uniform", 0.02), (40001, 262144 + 4097, 3, "uniform", 0.03),
    (300001, 40961, 1, "uniform", 0.012), (1000003, 1000100, 4, "uniform", 0.092),
])
def test_ordered_sums(ctx, formula, E, M, N, D, data, sigma):
    if formula == "gauss_gradx" and D == 4:
        pytest.skip("the fused gradient's fast path has D <= 3")
    rng = np.random.default_rng(M)
    x, y = _clouds(rng, M, N, D, data)
    x[7] = 1.2                                   # a row far from its neighbours on the curve
    assert _ordered(x, y, 1.4426950408889634 / (2 * sigma * sigma))
    b = rng.standard_normal((N, E)).astype(np.float32)
    b[np.linalg.norm(y - x[11], axis=1) < 2 * sigma] = 0      # a row whose near sum is zero
    red = "lse" if formula == "sinkhorn" else "sum"
    kw = dict(sigma=sigma, eps=2 * sigma * sigma)
    dx, dy, db = dev(x), dev(y), dev(b)
    got = host(ctx.run(formula, red, dx, dy, db, **kw))
    rows = np.unique(np.concatenate([[7, 11], _rows(rng, M, 64)]))
    place = host(ctx.run(formula, red, dx, dy, db, col_blocks=2, **kw))
    if formula == "sinkhorn":
        ref, m = oracle.sinkhorn_lse(x, y, b, kw["eps"], rows=rows)
        assert lse_err(got[rows], ref, m) <= LSE_TOL
        # the exponent's error bound, 1.2e-4 log2 units on either side at c R^2 = 2048 (the
        # reference enters the two calls' products at different values), in proportion
        half = (np.maximum(x.max(0), y.max(0)) - np.minimum(x.min(0), y.min(0))) / 2
        L = 1.4426950408889634 / (2 * sigma * sigma) * float((half ** 2).sum())
        assert np.abs(got - place).max() <= 2e-5 + 2 * 1.2e-4 * np.log(2) * L / 2048
        return
    if formula == "gauss_gradx":
        a, g, norm, _ = _gradx(x, y, b, sigma, rows)
        assert norm_err(got[rows, 0], a, norm) <= SUM_TOL
        assert np.abs(sigma * (got[rows, 1:] - g) / np.maximum(norm, 1e-30)[:, None]).max() <= SUM_TOL
    else:
        ref, norm = oracle.kernel_sum("gauss", x, y, b, sigma=sigma, rows=rows)
        assert norm_err(got[rows], ref, norm) <= SUM_TOL
    # both sum the same terms in another order; each order's rounding is a few
    # 2^-24 of the normaliser, which the sum with |b| bounds
    cap = host(ctx.run("gauss", "sum", dx, dy, dev(np.abs(b)), col_blocks=2, sigma=sigma)).max(1)
    assert np.abs(got[:, 0] - place[:, 0]).max() <= 1e-5 * cap.max()
    assert np.all(np.abs(got[:, 0] - place[:, 0]) <= 1e-5 * cap + 1e-37)


def _gradx(x, y, b, sigma, rows):
    r = oracle.gauss_gradx(x, y, b, sigma, rows=rows)
    out, norm = r[0], r[1]
    return out[:, 0], out[:, 1:], norm[:, 0], None


@pytest.mark.parametrize("low", [-1.0e30, -3.0e38])
def test_ordered_log_sums_of_masked_columns(ctx, low):
    """The lowest weights on most columns (a mask): only the rest counts, whatever comes first."""
    rng = np.random.default_rng(5)
    x, y = _clouds(rng, 100001, 100130, 3, "uniform")
    g = rng.standard_normal((100130, 1)).astype(np.float32)
    g[100:] = low
    got = host(ctx.run("sinkhorn", "lse", dev(x), dev(y), dev(g), eps=0.002))
    rows = _rows(rng, 100001, 64)
    ref, m = oracle.sinkhorn_lse(x, y[:100], g[:100], 0.002, rows=rows)
    assert lse_err(got[rows], ref, m) <= LSE_TOL


# with the order and the all-pairs kernels' scratch behind it, the order
# alone (the kernels behind pack 80 bytes a column), points in place (more rows than the
# order has room for)
@pytest.mark.parametrize("M,N,K,fits", [(1500, 20000, 4, True), (1500, 450000, 10, False), (2200000, 3000, 4, False),
                                        (2200000, 3000, 1, False)])
def test_small_scratch_lists(ctx, M, N, K, fits):
    """The no-allocation entry point keeps taking calls whose scratch has no room for all of the order's."""
    rng = np.random.default_rng(6)
    x = rng.integers(0, 20, (M, 3)).astype(np.float32)
    y = rng.integers(0, 20, (N, 3)).astype(np.float32)
    need = kred.scratch_bytes("sqdist", "argkmin", M, N, 3, 0, K=K)
    assert (need < kred.NOALLOC_SCRATCH_BYTES - (1 << 20)) == fits
    got = host(ctx.run_noalloc("sqdist", "argkmin", dev(x), dev(y), K=K))
    rows = _rows(rng, M)
    assert np.array_equal(got[rows], oracle.argkmin(x, y, K, rows=rows)[0])


# the order (D = 3) and the 32x32-tile operands (D = 10) do not fit, the form without them does
@pytest.mark.parametrize("M,N,D,sigma", [(2200000, 5000, 3, 0.05), (300000, 20000, 10, 2.5)])
def test_small_scratch_sums(ctx, M, N, D, sigma):
    rng = np.random.default_rng(7)
    x, y = _clouds(rng, M, N, D, "mixture")
    b = rng.standard_normal((N, 1)).astype(np.float32)
    assert kred.scratch_bytes("gauss", "sum", M, N, D, 1, sigma=sigma) > kred.NOALLOC_SCRATCH_BYTES
    got = host(ctx.run_noalloc("gauss", "sum", dev(x), dev(y), dev(b), sigma=sigma))
    rows = _rows(rng, M, 64)
    ref, norm = oracle.kernel_sum("gauss", x, y, b, sigma=sigma, rows=rows)
    assert norm_err(got[rows], ref, norm) <= SUM_TOL


def test_order_repeats_under_graph_replay(ctx):
    import torch
    rng = np.random.default_rng(7)
    x, y = _clouds(rng, 30000, 30001, 3, "mixture")
    dx, dy = dev(x), dev(y)
    want = ctx.run("sqdist", "argkmin", dx, dy, K=10)
    out = torch.empty_like(want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.run("sqdist", "argkmin", dx, dy, out=out, K=10, stream=torch.cuda.current_stream())
    for _ in range(4):
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("D", [1, 3, 4])
@pytest.mark.parametrize("real", [3, 70, 4000])
def test_lists_leave_out_overflown_distances(ctx, D, real):
    """A column whose squared distance is beyond fp32 is in no list, as in the direct form; the
    lists of a row with fewer than K others end in -1."""
    rng = np.random.default_rng(real)
    M, N, K = 4200, 4300, 10
    x = rng.integers(0, 30, (M, D)).astype(np.float32)
    y = rng.integers(0, 30, (N, D)).astype(np.float32)
    far = rng.permutation(N)[real:]
    y[far] = np.where(rng.random((N - real, 1)) < 0.5, -1, 1) * np.float32(1e25)
    got = _lists(ctx, x, y, K)
    want = host(ctx.run("sqdist", "argkmin", dev(x), dev(y), K=K, flags=kred.FLAG_DIRECT))
    assert np.array_equal(got, want)
    assert not np.isin(got, far).any() and (real >= K or (got[:, real:] == -1).all())


def _us(f, n=5):
    import torch
    f()
    each = []
    for _ in range(n):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        f()
        e1.record()
        e1.synchronize()
        each.append(e0.elapsed_time(e1) * 1e3)
    return sorted(each)[n // 2]


@pytest.mark.parametrize("case", ["one far", "far clusters", "heavy tails"])
def test_order_of_unevenly_spread_points(ctx, case):
    """The order separates near points though the box holds them in few cells of an even grid: the lists
    are right, and their time stays near that of the same cloud alone (measured: up to 2.5 times; 20
    times where all points share a few cells)."""
    rng = np.random.default_rng(8)
    M = N = 100000
    x, y = _clouds(rng, M, N, 3, "mixture")
    plain = [dev(x), dev(y)]
    if case == "one far":
        x[7], y[9] = 1000, -700
    elif case == "far clusters":
        x[::2] += 30000
        y[::2] += 30000
    else:
        x, y = (np.exp(6 * rng.standard_normal((n, 3))).astype(np.float32) for n in (M, N))
    rows = _rows(rng, M, 64)
    got = _lists(ctx, x, y, 4)[rows]
    _, d = oracle.argkmin(x, y, 4, rows=rows)
    mine = ((x[rows, None].astype(np.float64) - y[got].astype(np.float64)) ** 2).sum(-1)
    assert np.all(np.abs(mine - d) <= 8 * 2.0 ** -24 * d + 1e-44)
    spread = [dev(x), dev(y)]
    t0, t1 = (_us(lambda: ctx.run("sqdist", "argkmin", *p, K=4)) for p in (plain, spread))
    assert t1 <= 7 * t0, (t1, t0)


@pytest.mark.parametrize("M,N,D", [(32768, 32768, 3), (32769, 600, 4), (131072, 131072, 3), (131073, 700, 3),
                                   (700, 131073, 1), (65536, 2049, 2), (65537, 2048, 2)])
def test_lists_around_the_sorts_forms(ctx, M, N, D):
    """Two and three passes, prefixes by the scatter and by a kernel of their own."""
    rng = np.random.default_rng(M + N + D)
    x = rng.integers(0, 50, (M, D)).astype(np.float32)
    y = rng.integers(0, 50, (N, D)).astype(np.float32)
    rows = _rows(rng, M)
    assert np.array_equal(_lists(ctx, x, y, 12)[rows], oracle.argkmin(x, y, 12, rows=rows)[0])


def _shell(rng, N, top):
    """Integer points at one distance of the origin (many times each)."""
    g = np.arange(-top, top + 1)
    v = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    n = (v ** 2).sum(1)
    best = max(set(n.tolist()), key=lambda s: (n == s).sum())
    v = v[n == best]
    return v[rng.integers(0, len(v), N)].astype(np.float32)


# rows inside a shell of columns: the order cannot keep any column out, and the rows
# are left to the kernels that visit every pair (both row-block sizes, with and without
# a second pass; sparse rows of that kind among others; K beyond 16 stays)
@pytest.mark.parametrize("M,N,K,scale,some", [
    (16384, 20000, 1, 1, False), (16500, 20001, 10, 1, False), (16500, 20001, 4, 1, True), (3000, 20000, 10, 1, False),
    (16500, 20001, 16, 1, True), (16500, 20001, 10, 60, False), (140001, 9000, 10, 1, True), (2100, 20000, 30, 1, False),
    (700001, 8300, 2, 1, True), (16500, 20001, 1, 60, True),
])
@pytest.mark.parametrize("reduction", ["argkmin", "kmin"])
def test_lists_that_the_order_does_not_help(ctx, M, N, K, scale, some, reduction):
    rng = np.random.default_rng(M + K)
    y = _shell(rng, N, 12) * scale
    x = rng.integers(-1, 2, (M, 3)).astype(np.float32) * scale
    if some:
        x[np.arange(M) % 977 != 5] += np.float32(9 * scale)
    rows = np.unique(np.concatenate([_rows(rng, M), np.arange(5, M, 977)[:40]]))
    got = _lists(ctx, x, y, K, reduction)[rows]
    want, d = oracle.argkmin(x, y, K, rows=rows)
    assert np.array_equal(got, want if reduction == "argkmin" else d.astype(np.float32))


@pytest.mark.parametrize("M,N,K", [(16500, 20001, 10), (40000, 30011, 1), (3000, 20000, 40)])
def test_lists_of_many_equal_points(ctx, M, N, K):
    """A third of both clouds at one place (padding): the lowest indices of it, whatever the order."""
    rng = np.random.default_rng(M)
    x = rng.integers(0, 60, (M, 3)).astype(np.float32)
    y = rng.integers(0, 60, (N, 3)).astype(np.float32)
    x[::3] = 7
    y[1::3] = 7
    rows = _rows(rng, M)
    assert np.array_equal(_lists(ctx, x, y, K)[rows], oracle.argkmin(x, y, K, rows=rows)[0])
    assert np.array_equal(_lists(ctx, x, y, K)[3], np.arange(N)[(y == 7).all(1)][:K])


def test_time_of_lists_that_the_order_does_not_help(ctx):
    """Not far behind the kernels that visit every pair (which the flag selects), nor where many
    points coincide.  Measured 1.15 times; 6 times when such rows were finished over the order."""
    rng = np.random.default_rng(4)
    s = rng.standard_normal((100000, 3))
    y = dev((s / np.linalg.norm(s, axis=1, keepdims=True)).astype(np.float32))
    x = dev((1e-4 * rng.uniform(0, 1, (100000, 3))).astype(np.float32))
    run = lambda flags: _us(lambda: ctx.run("sqdist", "argkmin", x, y, K=1, flags=flags))
    t0, t1 = run(kred.FLAG_FAST), run(0)
    assert t1 <= 2 * t0, (t1, t0)
    x, y = _clouds(rng, 100000, 100000, 3, "mixture")
    px, py = dev(x), dev(y)
    plain = _us(lambda: ctx.run("sqdist", "argkmin", px, py, K=10))
    x[::3] = 3
    y[::3] = 3
    px, py = dev(x), dev(y)
    t2 = _us(lambda: ctx.run("sqdist", "argkmin", px, py, K=10))
    assert t2 <= 2 * plain, (t2, plain)


@pytest.mark.parametrize("some", [False, True])
def test_way_back_repeats_under_graph_replay(ctx, some):
    """Every replay counts its own given up rows: all of them, or some among others."""
    import torch
    rng = np.random.default_rng(9)
    y = dev(_shell(rng, 20001, 12))
    x = rng.integers(-1, 2, (16500, 3)).astype(np.float32)
    if some:
        x[np.arange(16500) % 977 != 5] += 9
    x = dev(x)
    want = ctx.run("sqdist", "argkmin", x, y, K=10)
    out = torch.empty_like(want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.run("sqdist", "argkmin", x, y, out=out, K=10, stream=torch.cuda.current_stream())
    for _ in range(4):
        out.zero_()
        ctx.run("sqdist", "argkmin", y, x, K=3)      # other work on the same scratch
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
