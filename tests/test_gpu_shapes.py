"""GPU parity, bit for bit, at the sizes where a launch changes its shape or a
kernel its branch: edges of tiles and row slots, remainders, the smallest and
largest of a range.  The reference is the CPU oracle."""
import sys

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


def _fit_equal(g, r, tag):
    assert int(g["status"][0]) == 0, (tag, g["status"])
    assert int(g["j"][0]) == r["j"], tag
    assert g["v"].tobytes() == r["v"].tobytes(), (tag, np.argwhere(g["v"] != r["v"])[:5])
    assert np.array_equal(g["row"], r["row"]), tag
    assert g["z_all"].tobytes() == r["z_all"].tobytes(), tag


def _path_equal(g, r, tag):
    assert int(g["status"][0]) == 0, (tag, g["status"])
    assert np.array_equal(g["J"], r["J"]), tag
    assert g["V"].tobytes() == r["V"].tobytes(), (tag, np.argwhere(g["V"] != r["V"])[:5])
    assert np.array_equal(g["ROW"], r["ROW"]), tag
    assert g["ZALL"].tobytes() == r["ZALL"].tobytes(), tag


def _data(seed, n, m, kind):
    if kind == "counts":
        return wl.random_small(seed, n, m, integer=True, zero_frac=0.3, span=4)
    if kind == "dense":
        return wl.accuracy_matrix(n, m, seed)[0]
    return wl.rank_one_matrix(n, m, max(1, m // 10), n // 10, 20.0, 0.01, (11, seed, n, m))


# row parts of the sign sums: one part, a last part of one row, an empty last
# part, the most parts, more than one tile each way
@pytest.mark.parametrize("n,m", [(63, 5), (129, 30), (1040, 64), (2049, 65), (2311, 7), (1025, 130)])
@pytest.mark.parametrize("kind", ["sparse", "counts"])
def test_sign_sum_row_parts(ctx, n, m, kind):
    from paper_2402_16712_amd import binding as B
    print(f"case parts {n}x{m} {kind}", flush=True)
    sys.stdout.flush()
    X = _data(n, n, m, kind)
    big = wl.max_column_mass(X)
    Xd = B.device_matrix(X)
    _fit_equal(_host(ctx.fit(Xd, 0.05 * big)), O.fit(X, 0.05 * big), (n, m, kind))
    lams = np.array([0.0, 0.01 * big, 0.3 * big])
    r = O.fit_path(X, lams)
    _path_equal(_host(ctx.fit_path(Xd, lams)), r, (n, m, kind))
    # a batch whose other problem is shorter than one part
    Y = _data(n + 1, 17, 9, kind)
    got = ctx.fit_batch([(Xd, lams), (B.device_matrix(Y), lams)])
    _path_equal(_host(got[0]), r, (n, m, kind, "batch"))
    _path_equal(_host(got[1]), O.fit_path(Y, lams), (n, m, kind, "batch"))


# the no-alloc workspace leaves room for all, some and none of the row parts
@pytest.mark.parametrize("m", [200, 700, 960])
def test_noalloc_row_parts(ctx, m):
    from paper_2402_16712_amd import binding as B
    print(f"case noalloc {m}", flush=True)
    X = _data(m, 700, m, "sparse")
    Xd, lam = B.device_matrix(X), 0.05 * wl.max_column_mass(X)
    a, b = _host(ctx.fit_noalloc(Xd, lam)), _host(ctx.fit(Xd, lam))
    for key in a:
        assert a[key].tobytes() == b[key].tobytes(), (m, key)


# the forms of the column preparation: column in LDS (one row to the longest),
# four waves from global memory, one wave per column; the last slots partial
@pytest.mark.parametrize("n,m", [(1, 2), (65, 3), (4096, 2), (4097, 3), (5003, 2), (70, 2100), (4200, 1030)])
def test_column_statistics_forms(ctx, n, m):
    from paper_2402_16712_amd import binding as B
    print(f"case columns {n}x{m}", flush=True)
    X = _data(n + m, n, m, "sparse")
    X[:, 0] *= 2.0 ** -60
    X[: n // 2, m - 1] = 0.0
    W, zeros, st = (t.cpu().numpy() for t in ctx.column_stats(B.device_matrix(X)))
    r = O.column_stats(X)
    assert int(st[0]) == 0
    assert W.tobytes() == np.asarray(r[0]).tobytes()
    assert np.array_equal(zeros, (X == 0.0).sum(axis=0))


# the division-free segment kernels at the edges of their row words (32 slots),
# of the window list, of the probe cuts and of the LDS copy of column j
@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 513, 2047, 2048, 2049, 2177, 3000, 4096, 4097, 6200, 9000])
@pytest.mark.parametrize("kind", ["sparse", "dense", "counts"])
def test_segment_rows(ctx, n, kind):
    from paper_2402_16712_amd import binding as B
    m = 9 if n < 3000 else 5
    print(f"case rows {n}x{m} {kind}", flush=True)
    X = _data(3 * n + 1, n, m, kind)
    big = max(wl.max_column_mass(X), 1.0)
    Xd = B.device_matrix(X)
    for lam in (0.0, 0.031 * big, 0.4 * big):
        _fit_equal(_host(ctx.fit(Xd, lam)), O.fit(X, lam), (n, kind, lam))
    lams = np.concatenate([big * 10.0 ** np.linspace(-4, 0, 9), [0.0]])
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, kind, "path"))


# one to three values: a whole bin of equal ratios, divided again by row
@pytest.mark.parametrize("n", [300, 2000, 4200, 9000])
@pytest.mark.parametrize("span", [1, 2])
def test_segment_ties(ctx, n, span):
    from paper_2402_16712_amd import binding as B
    print(f"case ties {n} span {span}", flush=True)
    X = wl.random_small(n + span, n, 5, integer=True, span=span)
    X[:, 4] = X[:, 0]                       # every ratio of a pair the same
    X[:, 3] *= 2.0 ** -20
    Xd = B.device_matrix(X)
    for lam in (0.0, 1.5, 7.0, 0.1 * n):
        _fit_equal(_host(ctx.fit(Xd, lam)), O.fit(X, lam), (n, span, lam))
    lams = np.array([7.0, 0.0, 0.1 * n, 1.5, 3.0])
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, span, "path"))


# penalties: one group of lanes, its last lane, a second group; unsorted; more
# distinct solutions than one residual pass scores
@pytest.mark.parametrize("L", [2, 5, 63, 64, 65, 128])
@pytest.mark.parametrize("n", [700, 5000])
def test_segment_penalties(ctx, L, n):
    from paper_2402_16712_amd import binding as B
    print(f"case penalties {L} rows {n}", flush=True)
    m = 12 if n < 1000 else 4
    X = _data(L + n, n, m, "sparse")
    lams = np.random.default_rng(L).permutation(wl.log_lambdas(wl.max_column_mass(X), L, -4.0))
    _path_equal(_host(ctx.fit_path(B.device_matrix(X), lams)), O.fit_path(X, lams), (L, n))


# columns outside the division-free range next to columns inside it, signed
# zeros, subnormals: the segments left to the exact kernel
@pytest.mark.parametrize("n", [130, 2100, 5000])
def test_segment_ranges(ctx, n):
    from paper_2402_16712_amd import binding as B
    print(f"case ranges {n}", flush=True)
    X = _data(n + 7, n, 7, "sparse")
    X[:, 1] *= 2.0 ** -420
    X[:, 2] *= 2.0 ** 380
    X[: n // 3, 3] = -0.0
    X[::5, 4] = 0.0
    X[:, 5] = np.sign(X[:, 5]) * 2.0 ** -300
    Xd = B.device_matrix(X)
    for lam in (0.0, 0.05 * wl.max_column_mass(X[:, :1]), 1e120):
        _fit_equal(_host(ctx.fit(Xd, lam)), O.fit(X, lam), (n, lam))
    lams = np.array([0.0, 1e-130, 1.0, 50.0, 1e115])
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, "path"))


# the feature sign sums in fragment order: one wave per workgroup (few output
# blocks) and four, partial fragments either way.  Bounds of the header, u = 2^-24
@pytest.mark.parametrize("n,m", [(1, 1), (33, 17), (130, 70), (257, 64), (45, 1500)])
def test_feature_sign_sums_layout(ctx, n, m):
    from paper_2402_16712_amd import binding as B
    print(f"case feature sums {n}x{m}", flush=True)
    X = _data(n + m, n, m, "sparse")
    X[: n // 3, m // 2] = 0.0
    DZ = ctx.feature_signsums(B.device_matrix(X)).cpu().numpy()
    W, u = np.abs(X).sum(axis=0), 2.0 ** -24
    D, Z = X.T @ np.sign(X), np.abs(X).T @ (X == 0.0)
    slack = n * 2.0 ** -52 * W[:, None]
    assert np.all(np.abs(DZ[:, :, 0] - D) <= (2.0 ** -15 + 2 * n * u) * W[:, None] + slack)
    assert np.all(np.abs(DZ[:, :, 1] - Z) <= (2.0 ** -8 + 2 * n * u) * Z + slack)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 2047, 2048, 2049, 2305])
@pytest.mark.parametrize("kind", ["sparse", "counts", "scaled", "wide"])
def test_breakpoint_counts(ctx, n, kind):
    # one pass over slots of 32 x 64 rows; minimisers of both signs and at 0,
    # columns whose magnitudes take the general branch ("scaled"), and a
    # column that is refused for its span unless its first row is 0 ("wide")
    from paper_2402_16712_amd import binding as B
    X = _data(900 + n, n, 6, kind if kind == "counts" else "sparse")
    X[:, 3] = -X[:, 2]
    if kind == "wide":
        X[:, 1] *= 2.0 ** -310
        X[0, 4] *= 2.0 ** 305
    if kind == "scaled":
        X[:, 1] *= 2.0 ** -310
        X[:, 4] *= 2.0 ** 305
    X = np.asfortranarray(X)
    print(f"case breakpoint counts n={n} {kind}", flush=True)
    g, r = _host(ctx.breakpoints(B.device_matrix(X))), O.breakpoints(X)
    if kind == "wide" and n > 1 and X[0, 4] != 0.0:
        assert int(g["status"][0]) == B.EWIDE
        return
    assert int(g["status"][0]) == 0
    assert np.array_equal(g["offsets"], r["offsets"])
    for key in ("lambda_max", "lam", "v"):
        assert g[key].tobytes() == r[key].tobytes(), key
    assert np.array_equal(g["row"], r["row"])


# work items of a batch: the fewest (two per workgroup), between, and the most
# per CU; more problems than XCDs and fewer.  Reference: each problem's own fit
@pytest.mark.parametrize("sizes", [[(5, 2)], [(150, 30)] * 9, [(500, 150), (60, 20), (300, 90)],
                                   [(2100, 200), (700, 40)], [(2000, 330), (1500, 210)]])
def test_batch_item_counts(ctx, sizes):
    from paper_2402_16712_amd import binding as B
    print(f"case batch items {sizes}", flush=True)
    probs = []
    for q, (n, m) in enumerate(sizes):
        X = _data(300 + q, n, m, ("sparse", "counts", "dense")[q % 3])
        probs.append((B.device_matrix(X), np.array([0.07 * wl.max_column_mass(X)])))
    for graph in (False, True, True):
        outs = ctx.fit_batch(probs, graph=graph)
        for (Xd, lam), o in zip(probs, outs):
            g, r = _host(o), _host(ctx.fit(Xd, float(lam[0])))
            assert int(g["status"][0]) == 0 == int(r["status"][0])
            assert int(g["J"].ravel()[0]) == int(r["j"][0])
            for a, b in (("V", "v"), ("ROW", "row"), ("ZALL", "z_all")):
                assert g[a].ravel().tobytes() == r[b].ravel().tobytes(), a


# whole numbers at whole penalties: targets that tie with prefix weights and
# sides that tie, columns of few and many rows, a unit other than 1
@pytest.mark.parametrize("n", [7, 64, 545, 2300, 5000])
@pytest.mark.parametrize("unit", [1.0, 2.0 ** -20])
def test_whole_penalties(ctx, n, unit):
    from paper_2402_16712_amd import binding as B
    print(f"case whole penalties n={n} unit={unit}", flush=True)
    X = np.asfortranarray(_data(700 + n, n, 9, "counts") * unit)
    Xd = B.device_matrix(X)
    top = wl.max_column_mass(X) / unit
    lams = unit * np.array([0.0, 1.0, 2.0, round(0.05 * top), round(0.05 * top) + 0.5, round(0.3 * top) + 1.0, top])
    for lam in lams:
        _fit_equal(_host(ctx.fit(Xd, float(lam))), O.fit(X, float(lam)), (n, lam))
    lams = np.unique(lams)
    _path_equal(_host(ctx.fit_path(Xd, lams)), O.fit_path(X, lams), (n, "path"))


def _correlated_counts(seed, n, m):
    """Whole numbers <= 60 whose rows and columns share a scale: v_k != 0 for
    most pairs, and hundreds to thousands of equal ratios."""
    g = np.random.default_rng(seed)
    scale = 0.6 * g.standard_normal(n)[:, None] + 0.6 * g.standard_normal(m)[None, :]
    return np.asfortranarray(np.minimum(np.floor(np.exp(scale) * 2.0 * g.random((n, m))), 60.0))


# several penalties: targets below the first window while the last of the others
# lie among more equal ratios than the list holds (seeds whose segments do so)
@pytest.mark.parametrize("n,L,seed", [(5000, 8, 2), (5000, 8, 3), (5000, 8, 4), (5000, 8, 6), (20000, 8, 5),
                                      (20000, 8, 9), (20000, 33, 2), (20000, 33, 3)])
def test_targets_below_a_tie(ctx, n, L, seed):
    from paper_2402_16712_amd import binding as B
    print(f"case below a tie {n} penalties {L} seed {seed}", flush=True)
    X = _correlated_counts(seed, n, 6)
    lams = wl.max_column_mass(X) * 10.0 ** (-3.0 + 3.0 * np.arange(L) / (L - 1))
    Xd, r = B.device_matrix(X), O.fit_path(X, lams)
    _path_equal(_host(ctx.fit_path(Xd, lams)), r, (n, L, seed))
    got = ctx.fit_batch([(Xd, lams), (Xd, lams[:1])])
    _path_equal(_host(got[0]), r, (n, L, seed, "batch"))
    _path_equal(_host(got[1]), O.fit_path(X, lams[:1]), (n, L, seed, "batch"))
