"""The exact segment kernel (what the division-free kernels leave): parity with
the CPU oracle in every form of its work list, and that its work spreads over
the chip, by times of the same process in ratio to each other."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2402_16712_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2402_16712_amd import binding as B
    c = B.Context(0)
    yield c
    c.close()


def _host(out):
    import torch
    torch.cuda.synchronize()
    return {k: (v.cpu().numpy() if v is not None else None) for k, v in out.items()}


def _path_equal(g, r, tag):
    assert int(g["status"][0]) == 0, (tag, g["status"])
    assert np.array_equal(g["J"], r["J"]), tag
    assert g["V"].tobytes() == r["V"].tobytes(), (tag, np.argwhere(g["V"] != r["V"])[:5])
    assert np.array_equal(g["ROW"], r["ROW"]), tag
    assert g["ZALL"].tobytes() == r["ZALL"].tobytes(), tag


def _matrix(n, m, seed):
    return wl.rank_one_matrix(n, m, max(1, m // 3), n // 10, 20.0, 0.01, (12, seed, n, m))


def _segment_ms(ctx, call):
    """Fastest of five runs of the segment kernels of one call."""
    import torch
    call()
    best = np.inf
    ctx.profile(True)
    try:
        for _ in range(5):
            ctx.profile_read(None, reset=True)
            call()
            torch.cuda.synchronize()
            best = min(best, ctx.profile_read("fit_seg", reset=True)[0])
    finally:
        ctx.profile(False)
    return best


# the columns at left are outside the division-free range: their segments are
# left as row or as column of the pair.  Words partly and wholly left, a last word
# of one segment, lists cut into eight, four and two pieces and not at all
@pytest.mark.parametrize("m,left", [(2, 2), (65, 65), (200, 200), (300, 7), (300, 300), (400, 3), (400, 50), (449, 449)])
def test_work_list_forms(ctx, m, left):
    from paper_2402_16712_amd import binding as B
    print(f"case work list {m} left {left}", flush=True)
    X = _matrix(70, m, left)
    big = wl.max_column_mass(X)
    X[:, np.random.default_rng(m).permutation(m)[:left]] *= 2.0 ** 990
    Xd = B.device_matrix(X)
    for lams in (np.array([0.05 * big]), np.array([0.0, 0.02 * big, 0.3 * big])):
        r = O.fit_path(X, lams)
        _path_equal(_host(ctx.fit_path(Xd, lams)), r, (m, left, len(lams)))
        got = ctx.fit_batch([(Xd, lams), (Xd, lams[:1])])
        _path_equal(_host(got[0]), r, (m, left, "batch"))


# residuals of one to eight distinct solutions per pass over the rows, a second
# pass, a second group of penalties
@pytest.mark.parametrize("L", [2, 3, 5, 7, 9, 17, 64, 65, 128])
def test_residuals_per_pass(ctx, L):
    from paper_2402_16712_amd import binding as B
    print(f"case residuals penalties {L}", flush=True)
    X = wl.accuracy_matrix(333, 9, L)[0] * 2.0 ** 950
    lams = wl.log_lambdas(wl.max_column_mass(X), L, -2.0)
    _path_equal(_host(ctx.fit_path(B.device_matrix(X), lams)), O.fit_path(X, lams), L)


# 552 segments are fewer than the chip's wave slots, so they take about as long
# as the slowest of them alone, here of eight pairs of columns at the same
# penalties (one after the other in 24 waves they took 23 times an average one;
# four times leaves room for what they share)
@pytest.mark.parametrize("L", [1, 8])
def test_few_segments_run_at_once(ctx, L):
    from paper_2402_16712_amd import binding as B
    print(f"case at once penalties {L}", flush=True)
    X = wl.accuracy_matrix(5000, 24, 3)[0] * 2.0 ** 950      # (dense direction: every v_k is nonzero)
    lams = 0.02 * wl.max_column_mass(X) * (1.0 + 0.3 * np.arange(L))
    Xd = B.device_matrix(X)
    many, two = _segment_ms(ctx, lambda: ctx.fit_path(Xd, lams)), 0.0
    for q in range(8):
        Xq = B.device_matrix(X[:, 3 * q:3 * q + 2])
        two = max(two, _segment_ms(ctx, lambda: ctx.fit_path(Xq, lams)))
    print(f"  552 segments {1e3 * many:.1f} us, 2 segments {1e3 * two:.1f} us", flush=True)
    assert many < 4.0 * two


def _correlated_counts(n, m, seed):
    g = np.random.default_rng(seed)
    scale = 0.6 * g.standard_normal(n)[:, None] + 0.6 * g.standard_normal(m)[None, :]
    return np.asfortranarray(np.minimum(np.floor(np.exp(scale) * 2.0 * g.random((n, m))), 60.0))


# whole numbers at whole penalties, where most targets tie with a prefix weight,
# take the route of the same numbers at penalties between whole ones (through
# the exact kernel they took 22 and 200 times as long)
@pytest.mark.parametrize("data", ["counts", "binary"])
def test_ties_at_several_penalties(ctx, data):
    from paper_2402_16712_amd import binding as B
    print(f"case ties at penalties {data}", flush=True)
    X = _correlated_counts(3000, 60, 5)
    if data == "binary":
        X = np.minimum(X, 1.0)
    whole = np.unique(np.round(wl.log_lambdas(wl.max_column_mass(X), 8, -3.0)))
    Xd = B.device_matrix(X)
    a, b = (_segment_ms(ctx, lambda lam=lam: ctx.fit_path(Xd, lam)) for lam in (whole, whole + 0.375))
    print(f"  8 whole penalties {1e3 * a:.1f} us, between them {1e3 * b:.1f} us", flush=True)
    assert a < 2.0 * b
    _path_equal(_host(ctx.fit_path(Xd, whole)), O.fit_path(X, whole), data)


# the edges of the unit: column sums just below and above 2^50 of them, units far
# from 1, penalties that vanish next to the unit, lie between two, or exceed all
@pytest.mark.parametrize("top", [2.0 ** 3, 2.0 ** 38, 2.0 ** 42])
@pytest.mark.parametrize("unit", [1.0, 2.0 ** -250, 2.0 ** 200])
def test_unit_edges(ctx, top, unit):
    from paper_2402_16712_amd import binding as B
    print(f"case unit edges {top} {unit}", flush=True)
    g = np.random.default_rng(int(np.log2(top)))
    u = g.standard_normal(1100)
    X = np.round((np.outer(u, g.standard_normal(8)) + 0.3 * g.standard_normal((1100, 8))) * top / 4.0)
    X[:, 3] = X[:, 1]
    X[::2, 3] += 1.0
    X[:, 6] = np.sign(X[:, 6])
    X[:, 7] = 0.0
    X = np.asfortranarray(X * unit)
    big = wl.max_column_mass(X)
    lams = np.concatenate([unit * np.array([1e-300, 0.25, 0.5, 1.0, 1.75, 3.0, 300.0, 300.5]), [0.0, 1e-307, 1e300],
                           unit * np.round(np.array([0.03, 0.2, 0.7]) * big / unit), [big]])
    Xd = B.device_matrix(X)
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (top, unit))
    for lam in lams:
        got = ctx.fit_batch([(Xd, np.array([lam]))])
        _path_equal(_host(got[0]), O.fit_path(X, [lam]), (top, unit, lam))


def _decimals(n, m, seed, places=1):
    return np.round(wl.accuracy_matrix(n, m, seed)[0], places)


# decimal fractions: ratios that differ in the last bits only, and equal ones, in
# lists of every length of the sort
@pytest.mark.parametrize("n", [90, 300, 700, 1500, 3300, 6000])
@pytest.mark.parametrize("places", [0, 1, 2])
def test_ratios_that_nearly_tie(ctx, n, places):
    from paper_2402_16712_amd import binding as B
    print(f"case near ties {n} places {places}", flush=True)
    X = _decimals(n, 10, n, places)
    X[:, 4] = 0.7 * X[:, 2]
    X[:, 8] = np.round(X[:, 2] / 3.0, places) * 3.0
    lams = wl.log_lambdas(wl.max_column_mass(X), 12, -3.0)
    lams[5] = np.round(lams[5])
    _path_equal(_host(ctx.fit_path(B.device_matrix(X), lams)), O.fit_path(X, lams), (n, places))


# rounded to one decimal, data take at most the five sorts more of their lists
# (through the exact kernel they took 13 times as long as unrounded)
def test_near_ties_stay_out_of_the_exact_kernel(ctx):
    from paper_2402_16712_amd import binding as B
    print("case near ties time", flush=True)
    X = wl.accuracy_matrix(1000, 100, 6)[0]
    lams = wl.log_lambdas(wl.max_column_mass(X), 16, -3.0)
    Xr, Xd = B.device_matrix(np.round(X, 1)), B.device_matrix(X)
    a, b = (_segment_ms(ctx, lambda A=A: ctx.fit_path(A, lams)) for A in (Xr, Xd))
    print(f"  rounded {1e3 * a:.1f} us, unrounded {1e3 * b:.1f} us", flush=True)
    assert a < 5.0 * b


# columns up to the edges of the division-free range and past them, alone and
# against each other: zeros of both signs, a column of one magnitude, subnormals
@pytest.mark.parametrize("n", [70, 600, 4200])
@pytest.mark.parametrize("scales", [(320, -420, 899, -880), (960, -960, 0, 500), (-885, -870, -200, -1040)])
def test_column_ranges(ctx, n, scales):
    from paper_2402_16712_amd import binding as B
    print(f"case column ranges {n} {scales}", flush=True)
    X = _matrix(n, 10, n)
    X += np.outer(np.random.default_rng(n).standard_normal(n), np.linspace(-1.0, 1.0, 10))
    X[:, 9] = np.sign(X[:, 9])
    X[::4, 2] = 0.0
    X[1::4, 2] = -0.0
    X[::5, 6] = 0.0
    for q, e in enumerate(scales):
        X[:, 2 * q] = np.ldexp(X[:, 2 * q], e)
        X[:, 2 * q + 1] = np.ldexp(X[:, 2 * q + 1], e)
    X = np.asfortranarray(X)
    Xd = B.device_matrix(X)
    for lam in [0.0] + [0.03 * wl.max_column_mass(X[:, q:q + 1]) for q in (0, 3, 5, 9)]:
        r = O.fit_path(X, [lam])
        g = _host(ctx.fit_path(Xd, np.array([lam])))
        if r["status"] != 0:                     # (a ratio that overflows is reported)
            assert int(g["status"][0]) == r["status"]
            continue
        _path_equal(g, r, (n, scales, lam))
    lams = np.sort([0.01 * wl.max_column_mass(X[:, q:q + 1]) for q in range(10)])
    r, g = O.fit_path(X, lams), _host(ctx.fit_path(Xd, lams))
    assert int(g["status"][0]) == r["status"]
    if r["status"] == 0:
        _path_equal(g, r, (n, scales, "path"))


# a matrix scaled by a power of two has the same ratios and takes as long (by
# the exact kernel, from 2^300 on, four to twenty times; twice leaves room for
# the times' spread)
@pytest.mark.parametrize("L", [1, 8])
def test_scaled_matrix_takes_as_long(ctx, L):
    from paper_2402_16712_amd import binding as B
    print(f"case scaled penalties {L}", flush=True)
    X = wl.accuracy_matrix(1500, 100, 8)[0]
    lams = 0.02 * wl.max_column_mass(X) * (1.0 + 0.3 * np.arange(L))
    X1, X2 = B.device_matrix(X), B.device_matrix(X * 2.0 ** 640)
    a, b = _segment_ms(ctx, lambda: ctx.fit_path(X2, lams * 2.0 ** 640)), _segment_ms(ctx, lambda: ctx.fit_path(X1, lams))
    print(f"  scaled {1e3 * a:.1f} us, unscaled {1e3 * b:.1f} us", flush=True)
    assert a < 2.0 * b


# breakpoint counts of pairs inside the division-free range and past it
@pytest.mark.parametrize("n", [1, 65, 700, 2305])
@pytest.mark.parametrize("e", [(320, -300), (490, -496), (950, 0), (-890, -905)])
def test_breakpoint_ranges(ctx, n, e):
    from paper_2402_16712_amd import binding as B
    print(f"case breakpoint ranges {n} {e}", flush=True)
    X = _matrix(n, 6, 40 + n)
    X[:, 3] = -X[:, 2]
    X[::7, 5] = 0.0
    X[:, 1] = np.ldexp(X[:, 1], e[0])
    X[:, 3] = np.ldexp(X[:, 3], e[0])
    X[:, 4] = np.ldexp(X[:, 4], e[1])
    X = np.asfortranarray(X)
    g, r = _host(ctx.breakpoints(B.device_matrix(X))), O.breakpoints(X)
    assert int(g["status"][0]) == 0
    assert np.array_equal(g["offsets"], r["offsets"])
    for key in ("lambda_max", "lam", "v"):
        assert g[key].tobytes() == r[key].tobytes(), key
    assert np.array_equal(g["row"], r["row"])


# a row that holds most of every column's weight is the solution of every segment
# and lies between equal samples; a window that has it inside settles the segment
# in one pass as any other (windows between the two samples missed it, and came
# to it after several)
@pytest.mark.parametrize("L", [1, 8])
def test_heavy_row(ctx, L):
    from paper_2402_16712_amd import binding as B
    print(f"case heavy row penalties {L}", flush=True)
    X = wl.accuracy_matrix(500, 200, 9)[0]
    Y = X.copy()
    Y[77] = 2.0 * np.abs(X).sum(axis=0) * np.where(X[77] < 0.0, -1.0, 1.0)
    lx, ly = (0.02 * wl.max_column_mass(A) * (1.0 + 0.3 * np.arange(L)) for A in (X, Y))
    Xd, Yd = B.device_matrix(X), B.device_matrix(Y)
    a, b = _segment_ms(ctx, lambda: ctx.fit_path(Yd, ly)), _segment_ms(ctx, lambda: ctx.fit_path(Xd, lx))
    print(f"  heavy {1e3 * a:.1f} us, without {1e3 * b:.1f} us", flush=True)
    assert a < 1.5 * b
    _path_equal(_host(ctx.fit_path(Yd, ly)), O.fit_path(Y, ly), L)


# an outlier repeated in a tenth of the rows: most samples are equal, and most of
# the other rows lie in the few gaps between them.  A gap's rows are listed in a
# few parts, so the segments take a few times what they take with outliers that
# differ (segments that ran out of windows took the exact kernel: 40 times)
@pytest.mark.parametrize("L", [1, 16])
def test_gaps_between_samples(ctx, L):
    from paper_2402_16712_amd import binding as B
    print(f"case gaps penalties {L}", flush=True)
    n = 5030
    g = np.random.default_rng(116)
    X = 0.1 * g.laplace(size=(n, 24)) + np.outer(g.standard_normal(n), g.standard_normal(24) * (g.random(24) < 0.3))
    rows = g.random(n) < 0.1
    Y = X.copy()
    X[rows] = 20.0 * g.standard_normal(24)
    Y[rows] = 20.0 * g.standard_normal((rows.sum(), 24))
    X, Y = np.asfortranarray(X), np.asfortranarray(Y)
    lx, ly = (wl.max_column_mass(A) * (10.0 ** np.linspace(-4.0, -1.0, 16))[8 if L == 1 else 0:][:L] for A in (X, Y))
    Xd, Yd = B.device_matrix(X), B.device_matrix(Y)
    a, b = _segment_ms(ctx, lambda: ctx.fit_path(Xd, lx)), _segment_ms(ctx, lambda: ctx.fit_path(Yd, ly))
    print(f"  1 outlier {1e3 * a:.1f} us, {rows.sum()} outliers {1e3 * b:.1f} us", flush=True)
    assert a < 5.0 * b
    _path_equal(_host(ctx.fit_path(Xd, lx)), O.fit_path(X, lx), L)


# columns of one magnitude that is no short binary fraction: sums of equal weights
# tie as whole numbers do, though none of them is exact
@pytest.mark.parametrize("n", [7, 64, 110, 1201, 5000])
@pytest.mark.parametrize("c", [0.1, 1.0 / 3.0 * 2.0 ** 700, np.nextafter(2.0 ** -890, 1.0)])
def test_columns_of_one_magnitude(ctx, n, c):
    from paper_2402_16712_amd import binding as B
    print(f"case one magnitude {n} {c}", flush=True)
    g = np.random.default_rng(n)
    u = g.standard_normal(n)
    X = np.sign(np.outer(u, g.standard_normal(9)) + 0.7 * g.standard_normal((n, 9))) * c
    X[:, 2] *= g.random(n) < 0.5
    X[:, 5] *= 3.0
    X[:, 6] = u * c                              # (all magnitudes, next to the others)
    X[:, 7] = 0.0
    X = np.asfortranarray(X)
    Xd = B.device_matrix(X)
    k = max(1, n // 20)
    steps = [0.0, c, np.nextafter(c, 0.0), 2.0 * c, k * c, np.nextafter(k * c, np.inf), 0.4 * n * c, 3.0 * n * c]
    for lam in steps:
        _path_equal(_host(ctx.fit_path(Xd, np.array([lam]))), O.fit_path(X, [lam]), (n, c, lam))
    lams = np.sort(np.array(steps))
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, c, "path"))


# at penalty 0 half of the segments of two-valued data tie: no longer than at one
# between two sums (twice leaves room for the times' spread; through the exact
# kernel three to eight times)
def test_one_magnitude_takes_as_long(ctx):
    from paper_2402_16712_amd import binding as B
    print("case one magnitude time", flush=True)
    g = np.random.default_rng(3)
    X = 0.1 * np.sign(np.outer(g.standard_normal(200), g.standard_normal(150)) + 0.5 * g.standard_normal((200, 150)))
    Xd = B.device_matrix(X)
    a, b = (_segment_ms(ctx, lambda lam=lam: ctx.fit(Xd, lam)) for lam in (0.0, 0.05))
    print(f"  penalty 0 {1e3 * a:.1f} us, between {1e3 * b:.1f} us", flush=True)
    assert a < 2.0 * b


# all rows of a bin of one ratio: ranked by counting up to 24 rows, sorted up to
# 64, divided again above; weights that differ, that tie and that are mixed
@pytest.mark.parametrize("n", [23, 24, 25, 26, 48, 50, 63, 64, 65, 100, 128, 130])
def test_equal_ratios(ctx, n):
    from paper_2402_16712_amd import binding as B
    print(f"case equal ratios {n}", flush=True)
    g = np.random.default_rng(n)
    X = g.standard_normal((n, 8))
    X[:, 1] = 0.5 * X[:, 0]
    X[:, 2] = -4.0 * X[:, 0]
    X[:, 3] = np.where(g.random(n) < 0.8, X[:, 0], 2.0 * X[:, 0])
    X[:, 4] = np.sign(X[:, 4])
    X[:, 5] = 3.0 * X[:, 4]
    X[:, 6] = np.where(g.random(n) < 0.7, X[:, 4], -X[:, 4])
    X = np.asfortranarray(X)
    Xd, big = B.device_matrix(X), wl.max_column_mass(X)
    for lam in (0.0, 1.0, 0.01 * big, 0.1 * big, 0.4 * big):
        _path_equal(_host(ctx.fit_batch([(Xd, np.array([lam]))])[0]), O.fit_path(X, [lam]), (n, lam))
    lams = big * 10.0 ** np.linspace(-3.0, -0.3, 7)
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, "path"))


# a column that is not finite: no route reads past the matrix (the padding below
# each column, changed between two calls, changes nothing) or gives a row past it
@pytest.mark.parametrize("n", [70, 130, 999, 4500])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_columns_not_finite(ctx, n, value):
    import torch
    print(f"case not finite {n} {value}", flush=True)
    g = np.random.default_rng(n)
    m, ld = 6, n + 320
    X = np.outer(g.standard_normal(n), g.standard_normal(m)) + 0.3 * g.standard_normal((n, m))
    X[:, 1] *= 2.0 ** 200
    X[::2, m - 2] = value                  # half of the samples of every other column
    X[int(np.argmax(np.abs(X[:, 0]))), m - 1] = value
    outs = []
    for fill in (0.0, 1.0, -1e30):
        buf = torch.full((m, ld), fill, dtype=torch.float64, device="cuda:0")
        buf[:, :n] = torch.from_numpy(np.ascontiguousarray(X.T)).cuda()
        Xd = buf.t()[:n]
        big = float(np.abs(X[:, 0]).sum())
        lams = np.concatenate(([0.0], big * 10.0 ** np.linspace(-3.0, -0.1, 6)))
        got = [_host(ctx.fit(Xd, lam)) for lam in lams] + [_host(ctx.fit_path(Xd, lams)), _host(ctx.breakpoints(Xd))]
        for d in got:
            assert int(d["status"].reshape(-1)[0]) != 0
            for key in ("median_row", "ROW"):
                if d.get(key) is not None:
                    assert int(d[key].max(initial=-1)) < n, key
        outs.append([{k: v.tobytes() for k, v in d.items() if v is not None and k in
                      ("v", "j", "obj", "median_row", "z_all", "V", "J", "OBJ", "ROW", "ZALL", "offsets")} for d in got])
    assert outs[0] == outs[1] == outs[2]
