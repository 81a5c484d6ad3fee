"""fp32 assignment on the fp16 matrix cores (csrc/split.hip, few tiles: csrc/split_small.hip): tile edges, odd sizes, and the
inputs that go back to the fp32 kernel (whole calls by their centroids, single tiles by their points).

Score bound: a dot product is rounded 6 times per 16 dims, each time by at most 2^-23 of a partial sum
(<= ||x|| ||c||), the split leaves out 3 2^-22 ||x|| ||c||, and ||c||^2 and the score are rounded to fp32.
"""
import numpy as np
import pytest

from gpu_util import NEAR_TIE_REL, host, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return torch_cuda()


@pytest.fixture(scope="module")
def km(torch):
    import paper_2608_14648_amd as m
    m.lib()
    return m


def points(n, d, k, seed, spread=0.2):
    g = np.random.default_rng(seed)
    C = g.standard_normal((k, d)).astype(np.float32)
    X = (C[g.integers(0, k, n)] + spread * g.standard_normal((n, d))).astype(np.float32)
    return X, C


def check(X, C, a, sc, rows=None):
    """a, sc against 64-bit scores on the given rows."""
    rows = np.arange(len(X)) if rows is None else rows
    Xd, Cd = X[rows].astype(np.float64), C.astype(np.float64)
    cn, xn = (Cd ** 2).sum(1), (Xd ** 2).sum(1)
    s = cn - 2 * (Xd @ Cd.T)
    got, best = a[rows], s.argmin(1)
    assert got.min() >= 0 and got.max() < len(C)
    i = np.arange(len(rows))
    gap = (s[i, got] - s[i, best]) / np.maximum(xn + np.maximum(cn[got], cn[best]), 1e-300)
    assert gap.max() <= NEAR_TIE_REL, gap.max()
    steps = 6 * -(-X.shape[1] // 16)
    xc = np.sqrt(xn * cn[got])
    bound = 2 * (steps * 2.0 ** -23 + 3 * 2.0 ** -22) * xc + 2.0 ** -22 * (cn[got] + np.abs(s[i, got]))
    err = np.abs(sc[rows].astype(np.float64) - s[i, got])
    assert (err <= bound).all(), (err / bound).max()
    return xn + s[i, got]


def spread_rows(n, k, tiles, d=32):
    """Row numbers of a call that repeats n rows: as they are, up to 4 tiles of 64 x 64 per CU; past that, where short
    chains of tiles are left to the fp32 kernel; or to chains of four stages of 32 dims per CU and more, split_kernel's."""
    if tiles == "few":
        return np.arange(n)
    if tiles == "many":
        return np.arange(n + 256 * -(-4 * 256 // (4 * -(-k // 64)))) % n
    tc = 128 if k <= 128 else 256
    nct = -(-k // tc)

    def chain(npt):
        return min(-(-npt * g // 256) * -(-nct // g) for g in range(1, min(8, nct) + 1)) * -(-d // 32) * tc / 256
    npt = max(-(-n // 256), 4 * 256 // (4 * -(-k // 64)) + 1)
    while chain(npt) < 4:
        npt += 64
    return np.arange(256 * npt - 3) % n


few_and_many = pytest.mark.parametrize("tiles", ["few", "many", "split"])


# k around the 64-, 128- and 256-centroid tiles and the centroid-tile groups, n around the 256-point tile, d from the
# smallest split one (two stages of 16 dims) through ragged last stages
@pytest.mark.parametrize("n,d,k", [(1, 32, 1), (5, 36, 2), (255, 32, 127), (256, 48, 128), (257, 44, 129), (300, 100, 255),
                                   (513, 64, 257), (1000, 132, 513), (3000, 96, 1100), (700, 772, 300), (64, 2048, 40)])
@few_and_many
def test_edges(km, torch, n, d, k, tiles):
    X, C = points(n, d, k, n + d + k)
    i = spread_rows(n, k, tiles, d)
    a, sc, obj = km.kmeans_assign(km.points_f32(to_dev(X[i], torch)), to_dev(C, torch), objective=True)
    a, sc = host(a), host(sc)
    np.testing.assert_array_equal(a, a[i])
    np.testing.assert_array_equal(sc, sc[i])
    dist = check(X, C, a[:n], sc[:n])[i]
    X = X[i]
    # summed from the distances: fp32 squares of fp32 differences, fp64 sums
    assert abs(host(obj)[0] - dist.sum()) <= 2.0 ** -20 * dist.sum() + 1e-12 * (X.astype(np.float64) ** 2).sum()


@few_and_many
def test_smallest_index_wins(km, torch, tiles):
    """Equal centroids in other blocks, lane halves, wave halves, tiles and groups of the sweep."""
    n, d, k = {"few": 700, "many": 5000, "split": 50000}[tiles], 64, 1300
    X, C = points(n, d, k, 3, spread=0.0)
    for src, copies in {5: (9, 37, 133, 300, 1299), 64: (68, 200, 700), 250: (251, 255, 513)}.items():
        C[list(copies)] = C[src]
    X[:300] = C[[5, 64, 250] * 100]
    a, _, _ = km.kmeans_assign(km.points_f32(to_dev(X, torch)), to_dev(C, torch))
    np.testing.assert_array_equal(host(a)[:300], [5, 64, 250] * 100)


@pytest.mark.parametrize("how", ["tiny_centroid", "zero_centroid", "wide_centroids", "huge", "small", "far_points"])
@pytest.mark.parametrize("k", [60, 300])
@few_and_many
def test_ranges(km, torch, how, k, tiles):
    """Scales at and past the ends of what the split takes: results keep the fp32 kernel's bound."""
    n, d = 900, 96
    X, C = points(n, d, k, 11)
    if how == "tiny_centroid":      # 2^-12 of the others: the fp32 kernel takes the call
        C[7] *= np.float32(2.0 ** -12)
        X[::9] = C[7] * np.float32(1.25)
    elif how == "zero_centroid":    # its products are exact
        C[7] = 0
        X[::9] *= np.float32(2.0 ** -10)
    elif how == "wide_centroids":   # within 2^-8
        C[::3] *= np.float32(2.0 ** -5)
        X[::9] = C[3] * np.float32(1.25)
    elif how == "huge":
        X, C = X * np.float32(2.0 ** 55), C * np.float32(2.0 ** 55)
    elif how == "small":
        X, C = X * np.float32(2.0 ** -55), C * np.float32(2.0 ** -55)
    else:                           # past fp16's range at the centroids' scale: their tile goes to the fp32 kernel
        X[300] *= np.float32(2.0 ** 14)
        X[301] *= np.float32(2.0 ** 7)
    i = spread_rows(n, k, tiles, d)
    a, sc, obj = km.kmeans_assign(km.points_f32(to_dev(X[i], torch)), to_dev(C, torch), objective=True)
    dist = check(X, C, host(a)[:n], host(sc)[:n])[i]
    X = X[i]
    assert abs(host(obj)[0] - dist.sum()) <= 2.0 ** -20 * dist.sum() + 1e-12 * (X.astype(np.float64) ** 2).sum()


@pytest.mark.parametrize("k", [60, 300, 2600])
@few_and_many
def test_not_finite(km, torch, k, tiles):
    """Rows with NaN or infinities: they answer as in the fp32 kernel and leave the others alone; the objective is NaN."""
    n, d = {"few": 3000, "many": 70000, "split": 300000}[tiles], 64
    if k == 2600:
        n = {"few": 1500, "many": 3000, "split": 30000}[tiles]
    X, C = points(max(n, k), d, k, 5)
    X = X[:n].copy()
    X[260, 3], X[700, 63] = np.nan, np.inf
    P = km.points_f32(to_dev(X, torch))
    a, sc, obj = km.kmeans_assign(P, to_dev(C, torch), objective=True)
    a, sc = host(a), host(sc)
    check(X, C, a, sc, np.setdiff1d(np.arange(n), [260, 700]))
    assert a[260] == np.iinfo(np.int32).max and sc[260] == np.inf  # no score is smaller than the start's
    assert a[700] == np.nonzero(C[:, 63] > 0)[0][0] and sc[700] == -np.inf
    assert np.isnan(host(obj)[0])
    if k <= n:
        Cn, _, J = km.kmeans_fit(P, k, 1, C=to_dev(C, torch))  # the fit's objective comes from its update
        assert np.isnan(host(J)).all()
    C[k // 2, 1] = np.nan  # a centroid with NaN never wins
    a, _, _ = km.kmeans_assign(P, to_dev(C, torch))
    assert not (host(a) == k // 2).any()


@pytest.mark.parametrize("how,want", [("no_centroid", np.inf), ("no_centroid_and_nan", np.nan), ("centroid", np.nan)])
@few_and_many
def test_objective_of_infinite_rows(km, torch, how, want, tiles):
    """An infinite coordinate for which every score is +infinity makes every objective +infinity (of a call, of a fit's
    updates and last pass, of FINE with and without an update), NaN beside it NaN; a score of -infinity NaN."""
    n, d, k = {"few": 900, "many": 70000, "split": 300000}[tiles], 64, 90
    X, C = points(n, d, k, 21)
    X[:, 0], C[:, 0] = -np.abs(X[:, 0]), -np.abs(C[:, 0]) - 0.1
    if how == "centroid":
        X[n // 2, 0] = -np.inf
    else:
        X[n // 2, 0] = np.inf
    if how == "no_centroid_and_nan":
        X[n // 3, 5] = np.nan
    P, Ct = km.points_f32(to_dev(X, torch)), to_dev(C, torch)
    a, _, J = km.kmeans_assign(P, Ct, objective=True)
    assert (host(a)[n // 2] < k) == (how == "centroid")
    np.testing.assert_array_equal(host(J), [want])
    if how != "centroid":  # (a centroid that takes an infinity is infinite after the update)
        _, _, J = km.kmeans_fit(P, k, 2, C=Ct.clone())
        np.testing.assert_array_equal(host(J), [want] * 3)
        meso = to_dev(np.where(np.arange(n) == 3, -1, np.arange(n) % 3).astype(np.int32), torch)
        for iters in (0, 1):
            _, _, _, J = km.kmeans_fine(P, meso, 3, k, iters, C=Ct.clone(), policy=km.KM_EMPTY_KEEP, objective=True)
            np.testing.assert_array_equal(host(J), [want])


@few_and_many
def test_objective_near_the_end_of_fp32(km, torch, tiles):
    """Squared distances of 2^127.4 each, in a call and in a fit's update: their sums are past fp32's range."""
    n, d, k = {"few": 900, "many": 70000, "split": 300000}[tiles], 64, 3
    g = np.random.default_rng(2)
    X, C = g.standard_normal((n, d)).astype(np.float32), g.standard_normal((k, d)).astype(np.float32)
    X[:, 0], C[:, 0] = 1.5e19 * g.choice([-1, 1], n), 0
    C[:, 1] = np.arange(k)
    P = km.points_f32(to_dev(X, torch))
    for J in (km.kmeans_assign(P, to_dev(C, torch), objective=True)[2], km.kmeans_fit(P, k, 1, C=to_dev(C, torch))[2]):
        np.testing.assert_allclose(host(J)[0], n * float(X[0, 0]) ** 2, rtol=1e-6)


def test_one_stage(km, torch):
    """Fewer dims than a stage of few tiles, odd and even numbers of stages, points with a stride."""
    for n, d, k in ((130, 32, 70), (65, 64, 64), (64, 68, 65), (200, 100, 1)):
        X, C = points(n, d, k, d)
        wide = torch.full((n, d + 12), float("nan"), device="cuda")
        wide[:, :d] = to_dev(X, torch)
        a, sc, _ = km.kmeans_assign(km.Points(km.KM_F32, wide[:, :d], d), to_dev(C, torch))
        check(X, C, host(a), host(sc))


def test_fit_objective(km, torch):
    """Every pass's objective (from the update that follows it, the last one directly) against 64 bits, with rows
    that have a stride and with the last update from raw rows."""
    n, d, k, T = 5000, 68, 90, 3
    X, C = points(n, d, k, 8, spread=1.0)
    wide = torch.zeros((n, 80), device="cuda")
    wide[:, :d] = to_dev(X, torch)
    raw = to_dev(X[::-1], torch)
    for Xt, r in ((to_dev(X, torch), None), (wide[:, :d], None), (to_dev(X, torch), raw)):
        P = km.Points(km.KM_F32, Xt, d, raw=r)
        _, _, J = km.kmeans_fit(P, k, T, C=to_dev(C, torch))
        Ct, want = C.astype(np.float64), []
        for t in range(T + 1):
            s = (Ct ** 2).sum(1) - 2 * (X.astype(np.float64) @ Ct.T)
            a = s.argmin(1)
            want.append(((X - Ct[a]) ** 2).sum())
            src = X[::-1] if r is not None and t == T - 1 else X
            for j in range(k):
                if (a == j).any():
                    Ct[j] = src[a == j].astype(np.float64).mean(0)
        np.testing.assert_allclose(host(J), want, rtol=1e-5)


def test_noalloc_past_its_scratch(km, torch):
    """A split image of 80 MB does not fit the static 64 MiB: the call is taken by the fp32 kernel, as before."""
    n, d, k = 300, 1024, 20000
    X, C = points(n, d, k, 2)
    P, Ct = km.points_f32(to_dev(X, torch)), to_dev(C, torch)
    a = torch.empty(n, dtype=torch.int32, device="cuda")
    sc = torch.empty(n, device="cuda")
    km.kmeans_assign_noalloc(P, Ct, a, sc)
    b, _, _ = km.kmeans_assign(P, Ct)
    np.testing.assert_array_equal(host(a), host(b))


# the tail's stages of 128 dims whole and partial, front of 2 stages and more, tiles of 128 and 256 centroids, groups
@pytest.mark.parametrize("n,d,d0,k", [(1, 64, 32, 1), (257, 96, 32, 128), (300, 160, 64, 129), (513, 288, 96, 300),
                                      (700, 704, 64, 257), (1500, 1024, 384, 1100)])
@pytest.mark.parametrize("how", ["plain", "tiny_centroid", "not_finite"])
def test_hybrid(km, torch, n, d, d0, k, how):
    """Front dims plus 1-bit tail against the 64-bit scores of the same codes."""
    import oracle as orc
    X, C = points(n, d, k, n + d0)
    if how == "tiny_centroid":  # the front of one centroid 2^-12 of the others: the fp32 kernel takes the call
        C[0, :d0] *= np.float32(2.0 ** -12)
        X[::9, :d0] = C[0, :d0] * np.float32(1.25)
    m = orc.col_mean(X)
    bits, alpha = orc.sign1_encode(X, m, d0)
    front = np.ascontiguousarray(X[:, :d0])
    bad = []
    if how == "not_finite":
        front[n // 2, 1] = np.nan
        bad = [n // 2]
    P = km.points_hybrid(to_dev(front, torch), to_dev(bits.view(np.int32), torch), to_dev(alpha, torch),
                         to_dev(m, torch), d)
    a, sc, obj = km.kmeans_assign(P, to_dev(C, torch), objective=True)
    a, sc = host(a), host(sc)
    rows = np.setdiff1d(np.arange(n), bad)
    assert (a[bad] == np.iinfo(np.int32).max).all() and (sc[bad] == np.inf).all()
    r = C[:, d0:] - m[d0:]  # residual codes in fp32, as the interface defines them
    sg = np.where(np.abs(r).max(1) > 0, np.abs(r).max(1) / np.float32(127), np.float32(1)).astype(np.float32)
    q = np.clip(np.rint(r / sg[:, None]), -127, 127).astype(np.float64)
    b = ((bits[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1).reshape(n, -1)[:, d0:].astype(np.float64) * 2 - 1
    f, cf = front[rows].astype(np.float64), C[:, :d0].astype(np.float64)
    cn = (cf ** 2).sum(1)
    tail = sg.astype(np.float64) ** 2 * (q ** 2).sum(1) - 2 * alpha[rows, None] * sg.astype(np.float64) * (b[rows] @ q.T)
    s = cn - 2 * f @ cf.T + tail
    i = np.arange(len(rows))
    if len(rows) == 0:
        return
    got = a[rows]
    xn = (f ** 2).sum(1)
    size = xn + cn[got] + np.abs(tail).max(1)
    assert ((s[i, got] - s.min(1)) / size).max() <= NEAR_TIE_REL
    # the front's bound, the partial sums starting at the tail's score
    steps = 6 * (d0 // 16)
    bound = 2 * (steps * 2.0 ** -23 + 3 * 2.0 ** -22) * size
    assert (np.abs(sc[rows] - s[i, got]) <= bound).all()
    if bad:
        assert np.isnan(host(obj)[0])
    else:  # from the distances: fp32 squares of the front's differences, the tail's scores in fp32, fp64 sums
        want = (s[i, got] + xn + alpha.astype(np.float64) ** 2 * (d - d0)).sum()
        assert abs(host(obj)[0] - want) <= 2.0 ** -21 * size.sum()


def hybrid_scores(front, bits, alpha, C, m, d0):
    """64-bit scores of hybrid points and their tail part, ||x'||^2 and ||c'||^2."""
    r = C[:, d0:] - m[d0:]  # residual codes in fp32, as the interface defines them
    sg = np.where(np.abs(r).max(1) > 0, np.abs(r).max(1) / np.float32(127), np.float32(1)).astype(np.float32)
    q = np.clip(np.rint(r / sg[:, None]), -127, 127).astype(np.float64)
    b = ((bits[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1).reshape(len(bits), -1)[:, d0:].astype(np.float64) * 2 - 1
    f, cf = front.astype(np.float64), C[:, :d0].astype(np.float64)
    cn = (cf ** 2).sum(1)
    tail = sg.astype(np.float64) ** 2 * (q ** 2).sum(1) - 2 * alpha[:, None] * sg.astype(np.float64) * (b @ q.T)
    return cn - 2 * f @ cf.T + tail, tail, (f ** 2).sum(1), cn


# as above, the rows repeated to chains that split_kernel takes
@pytest.mark.parametrize("n,d,d0,k", [(257, 96, 32, 128), (300, 160, 64, 129), (513, 288, 96, 300), (700, 704, 64, 257),
                                      (600, 1024, 384, 1100), (255, 672, 32, 60)])
@pytest.mark.parametrize("how", ["plain", "tiny_centroid", "not_finite"])
def test_hybrid_many(km, torch, n, d, d0, k, how):
    import oracle as orc
    X, C = points(n, d, k, n + d0)
    if how == "tiny_centroid":
        C[0, :d0] *= np.float32(2.0 ** -12)
        X[::9, :d0] = C[0, :d0] * np.float32(1.25)
    m = orc.col_mean(X)
    bits, alpha = orc.sign1_encode(X, m, d0)
    front = np.ascontiguousarray(X[:, :d0])
    i = spread_rows(n, k, "split", d0)
    fr, bad = front[i], []
    if how == "not_finite":
        bad = [len(i) - 5]
        fr[bad, 1] = np.nan
    P = km.points_hybrid(to_dev(fr, torch), to_dev(bits[i].view(np.int32), torch), to_dev(alpha[i], torch),
                         to_dev(m, torch), d)
    a, sc, obj = km.kmeans_assign(P, to_dev(C, torch), objective=True)
    a, sc = host(a), host(sc)
    assert (a[bad] == np.iinfo(np.int32).max).all() and (sc[bad] == np.inf).all()
    ok = np.setdiff1d(np.arange(len(i)), bad)
    s, tail, xn, cn = hybrid_scores(front, bits, alpha, C, m, d0)
    got, r = a[ok], i[ok]
    size = xn[r] + cn[got] + np.abs(tail).max(1)[r]
    assert ((s[r, got] - s.min(1)[r]) / size).max() <= NEAR_TIE_REL
    assert (np.abs(sc[ok] - s[r, got]) <= 2 * (6 * (d0 // 16) * 2.0 ** -23 + 3 * 2.0 ** -22) * size).all()
    if bad:
        assert np.isnan(host(obj)[0])
    else:
        want = (s[r, got] + xn[r] + alpha.astype(np.float64)[r] ** 2 * (d - d0)).sum()
        assert abs(host(obj)[0] - want) <= 2.0 ** -21 * size.sum()


# A tile of 3 stages, the fewest there are (front of 32 dims, tail of one stage), in workgroups that sweep 8 and 16
# tiles of 256 centroids: their constants take turns in two places.
@pytest.mark.parametrize("d,k", [(64, 2048), (160, 4090)])
def test_hybrid_three_stages(km, torch, d, k):
    import oracle as orc
    n, d0 = 600, 32
    X, C = points(n, d, k, d)
    C[:, :d0] *= (1 + np.arange(k, dtype=np.float32) % 7)[:, None]  # norms that differ from tile to tile
    m = orc.col_mean(X)
    bits, alpha = orc.sign1_encode(X, m, d0)
    front = np.ascontiguousarray(X[:, :d0])
    i = np.arange(65536) % n  # 256 point tiles, one per CU: a workgroup sweeps every centroid tile
    P = km.points_hybrid(to_dev(front[i], torch), to_dev(bits[i].view(np.int32), torch), to_dev(alpha[i], torch),
                         to_dev(m, torch), d)
    a, sc, _ = km.kmeans_assign(P, to_dev(C, torch))
    a, sc = host(a), host(sc)
    np.testing.assert_array_equal(a, a[i])
    np.testing.assert_array_equal(sc, sc[i])
    s, tail, xn, cn = hybrid_scores(front, bits, alpha, C, m, d0)
    r, got = np.arange(n), a[:n]
    size = xn + cn[got] + np.abs(tail).max(1)
    assert ((s[r, got] - s.min(1)) / size).max() <= NEAR_TIE_REL
    assert (np.abs(sc[:n] - s[r, got]) <= 2 * (12 * 2.0 ** -23 + 3 * 2.0 ** -22) * size).all()


# one and several 256-point tiles, output tiles of 128 and 256 and several of them, ragged dims
@pytest.mark.parametrize("n,d,dout", [(1, 32, 4), (255, 36, 8), (257, 64, 128), (300, 100, 132), (1000, 260, 256),
                                      (513, 132, 600), (64, 4096, 36)])
@pytest.mark.parametrize("how", ["plain", "rows", "not_finite", "columns", "nan_basis"])
def test_project(km, torch, n, d, dout, how):
    """Y = (X - mean) W against 64 bits, each value bounded by its own row and column: also rows and columns of
    very different size, and rows that only the fp32 kernel can take."""
    g = np.random.default_rng(n + d)
    X = g.standard_normal((n, d)).astype(np.float32) * np.float32(0.3)
    m = (X.astype(np.float64).mean(0) if n > 1 else np.full(d, 0.1)).astype(np.float32)
    W = (g.standard_normal((d, dout)) / np.sqrt(d)).astype(np.float32)
    if how == "rows":
        X[::7] = m + (X[::7] - m) * np.float32(2.0 ** -18)
        X[3::7] = m
        X[5::7] *= np.float32(2.0 ** 10)
    elif how == "not_finite":
        X[n // 2, d // 2] = np.nan
        X[n // 3, 1] = np.inf
    elif how == "columns":
        W[:, ::3] *= np.float32(2.0 ** -30)
        W[:, 1] = 0
    elif how == "nan_basis":
        W[d // 2, dout // 2] = np.nan
    with np.errstate(invalid="ignore"):
        xc = (X - m).astype(np.float64)  # centred in fp32, as the interface's kernels do
        want = xc @ W.astype(np.float64)
    Y = host(km.pca_project(to_dev(X, torch), to_dev(m, torch), to_dev(W, torch))).astype(np.float64)
    fin = np.isfinite(want)
    np.testing.assert_array_equal(np.isnan(Y), np.isnan(want))
    np.testing.assert_array_equal(Y[~fin & ~np.isnan(want)], want[~fin & ~np.isnan(want)])
    size = np.sqrt(np.nansum(np.where(np.isfinite(xc), xc, 0) ** 2, 1))[:, None] * np.sqrt(np.nansum(W.astype(np.float64) ** 2, 0))
    bound = (6 * -(-d // 16) * 2.0 ** -23 + 2.0 ** -20) * size + 1e-40
    err = np.abs(Y[fin] - want[fin])
    assert (err <= bound[fin]).all(), (err / bound[fin]).max()


# the same where split_kernel takes few dims: two rounds of 256-point tiles, dims a stage of 16 does not divide
@pytest.mark.parametrize("n,d,dout", [(66000, 36, 8), (65600, 60, 100), (197000, 32, 36), (66000, 100, 132)])
@pytest.mark.parametrize("how", ["plain", "rows", "not_finite", "columns"])
def test_project_many(km, torch, n, d, dout, how):
    test_project(km, torch, n, d, dout, how)


@pytest.mark.parametrize("row", [0, 31, 69, 32, 255])
def test_project_one_small_row(km, torch, row):
    """One row whose centred values are 2^-24 of the others', alone in its tile, in either block of a wave: the split
    would keep 2^-37 of the others, so the row goes to the fp32 kernel, also where its uncentred values are large."""
    n, d, dout = 256, 128, 40
    g = np.random.default_rng(row)
    m = np.where(np.arange(d) < 16, 64, 0).astype(np.float32)
    X = (m + g.standard_normal((n, d)) * 2.0 ** 10).astype(np.float32)
    X[row] = m + np.where(m > 0, 0, 2.0 ** -14 * g.standard_normal(d)).astype(np.float32)
    W = (g.standard_normal((d, dout)) / 8).astype(np.float32)
    xc = (X[row] - m).astype(np.float64)
    Y = host(km.pca_project(to_dev(X, torch), to_dev(m, torch), to_dev(W, torch)))[row].astype(np.float64)
    size = np.linalg.norm(xc) * np.linalg.norm(W.astype(np.float64), axis=0)
    assert (np.abs(Y - xc @ W.astype(np.float64)) <= (6 * d // 16 * 2.0 ** -23 + 2.0 ** -20) * size).all()


@pytest.mark.parametrize("how", ["small_dims", "small_weights", "one_column"])
def test_project_dims_of_different_size(km, torch, how):
    """Half of the dims 2^-20 of the others, and outputs that live on them: each output bounded by its own terms, as
    fp32 products are (2^-24 each, and 6 roundings per 16 dims)."""
    n, d, dout = 700, 128, 72
    g = np.random.default_rng(4)
    s = np.where(np.arange(d) % 2, 2.0 ** -20, 1.0)
    X = (g.standard_normal((n, d)) * s).astype(np.float32)
    W = g.standard_normal((d, dout)) / 8
    if how == "small_dims":      # the large dims have no part in an output
        W[0::2] = 0
    elif how == "small_weights":  # all terms of the same size
        W /= s[:, None] * 2.0 ** 20
    else:
        W[0::2, 50] = 0
    W = W.astype(np.float32)
    Y = host(km.pca_project(to_dev(X, torch), torch.zeros(d, device="cuda"), to_dev(W, torch))).astype(np.float64)
    Xd, Wd = X.astype(np.float64), W.astype(np.float64)
    bound = (6 * d // 16 * 2.0 ** -23 + 2.0 ** -23) * (np.abs(Xd) @ np.abs(Wd))
    err = np.abs(Y - Xd @ Wd)
    assert (err <= bound).all(), (err / bound).max()


# one row to several splits and runs of 4096 rows, ragged stages of 16 rows, one to three 256-column blocks
@pytest.mark.parametrize("n,d", [(1, 4), (15, 36), (16, 256), (31, 260), (33, 512), (4111, 300), (20001, 516), (70000, 32)])
def test_cov(km, torch, n, d):
    """Covariance of columns whose sizes differ by 2^60, one of them constant, against 64 bits, each entry bounded by
    its own two columns.  A run is rounded 6 times per 16 of its 4096 rows: 2^-24 sqrt(1536) of the sum at random, 2^-19
    with room for eight of these."""
    g = np.random.default_rng(n + d)
    X = (g.standard_normal((n, d)) + 0.5 * g.standard_normal((n, 1))) * 2.0 ** g.integers(-30, 30, d) + 3
    X = X.astype(np.float32)
    X[:, d // 2] = 1e7
    mean, cov = (host(v) for v in km.pca_fit_cov(to_dev(X, torch)))
    xc = (X - mean).astype(np.float64)
    want = xc.T @ xc / n
    size = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    assert (np.abs(cov - want) <= 2.0 ** -19 * size + 2.0 ** -22 * np.abs(want)).all()
    np.testing.assert_array_equal(cov, cov.T)
    assert (cov[d // 2] == 0).all()


def test_cov_not_finite(km, torch):
    """A NaN or an infinity spoils its own row and column only."""
    X = np.random.default_rng(0).standard_normal((3000, 300)).astype(np.float32)
    clean = host(km.pca_fit_cov(to_dev(X, torch))[1])
    X[1500, 7], X[20, 280] = np.nan, np.inf
    cov = host(km.pca_fit_cov(to_dev(X, torch))[1])
    bad = np.zeros(300, bool)
    bad[[7, 280]] = True
    assert np.isnan(cov[bad]).all() and np.isnan(cov[:, bad]).all()
    np.testing.assert_array_equal(cov[~bad][:, ~bad], clean[~bad][:, ~bad])


# front dims of two stages and more, whole and ragged; 128- and 256-centroid tiles; the last tile's words past the mask row
@pytest.mark.parametrize("n,d,df,k", [(1, 64, 24, 2), (257, 96, 32, 128), (300, 128, 40, 129), (1000, 256, 96, 300),
                                      (700, 512, 256, 1000), (513, 48, 48, 70)])
@pytest.mark.parametrize("how", ["plain", "far_points", "tiny_centroid", "not_finite"])
def test_pruned(km, torch, n, d, df, k, how):
    """The pruned pass against its definition in 64 bits: a pair is dropped at d' when its partial distance exceeds
    tau r(d'); candidates within 1e-5 of a threshold may go either way."""
    X, C = points(n, d, k, n + df, spread=0.5)
    g = np.random.default_rng(1)
    if how == "far_points":
        X[::5] *= np.float32(2.0 ** 14)
    elif how == "tiny_centroid":
        C[0] *= np.float32(2.0 ** -12)
    elif how == "not_finite":
        X[n // 2, 1] = np.nan
    prev = g.integers(0, k, n).astype(np.int32)
    a, dist, obj, cnt = km.kmeans_assign_pruned(km.points_f32(to_dev(X, torch)), to_dev(C, torch), to_dev(prev, torch),
                                                d_front=df, objective=True, counters=True)
    a, dist = host(a), host(dist)
    Xd, Cd = X.astype(np.float64), C.astype(np.float64)
    part = np.cumsum((Xd[:, None, :] - Cd[None]) ** 2, 2)
    i = np.arange(n)
    tau, full = part[i, prev, -1], part[:, :, -1]
    alive, sure = np.ones((n, k), bool), np.ones((n, k), bool)  # in reach of the test, and clear of it
    passed = np.zeros(2)
    for D in range(df, d, 64):
        lim = (tau * (1 + 2.1 / np.sqrt(D)) ** 2 * D / d)[:, None]
        room = 1e-5 * ((Xd[:, None, :D] ** 2).sum(2) + (Cd[None, :, :D] ** 2).sum(2) + lim)
        with np.errstate(invalid="ignore"):
            alive &= part[:, :, D - 1] <= lim + room
            sure &= part[:, :, D - 1] <= lim - room
        if D == df:
            passed = np.array([(m.sum() - m[i, prev].sum()) for m in (sure, alive)])
    alive[i, prev] = sure[i, prev] = True
    ok = np.isfinite(tau)
    best = np.where(sure, full, np.inf).min(1)
    assert alive[i, a][ok].all()
    assert (full[i, a][ok] <= best[ok] * (1 + 1e-5) + 1e-9).all()
    np.testing.assert_allclose(dist[ok], full[i, a][ok], rtol=2e-5)
    if how != "not_finite" and df < d:
        assert cnt[0] == n * (k - 1) and passed[0] <= cnt[1] <= passed[1]
    elif df == d:
        assert cnt[0] == cnt[1] == 0
    else:
        assert a[n // 2] == prev[n // 2] and np.isnan(dist[n // 2])


# the same where split_kernel takes few front dims: many centroids, fronts a stage of 16 does not divide
@pytest.mark.parametrize("n,d,df,k", [(100, 128, 40, 2100), (64, 96, 24, 2200), (150, 48, 48, 1100)])
@pytest.mark.parametrize("how", ["plain", "far_points", "tiny_centroid", "not_finite"])
def test_pruned_many(km, torch, n, d, df, k, how):
    test_pruned(km, torch, n, d, df, k, how)


def test_less_scratch(km, torch, monkeypatch):
    """Calls whose split image is refused: the fp32 kernel's results."""
    n, d, k = 20000, 256, 1000
    X, C = points(n, d, k, 9)
    W = (np.random.default_rng(9).standard_normal((d, d)) / 16).astype(np.float32)
    Xt, Ct, Wt, zero = to_dev(X, torch), to_dev(C, torch), to_dev(W, torch), torch.zeros(d, device="cuda")
    monkeypatch.setenv("KMQ_FAIL_ALLOC", ">300000")  # past the fp32 kernels' 262400 and 176128 bytes, less than the split's
    Y = host(km.pca_project(Xt, zero, Wt)).astype(np.float64)
    a, sc, _ = km.kmeans_assign(km.points_f32(Xt), Ct)
    monkeypatch.setenv("KMQ_FAIL_ALLOC", ">500000")
    _, _, _, R = km.rabitq_encode(Xt[:5000].contiguous(), Wt, zero, want_rotated=True)
    monkeypatch.delenv("KMQ_FAIL_ALLOC")
    check(X, C, host(a), host(sc), np.arange(500))
    want = X.astype(np.float64) @ W.astype(np.float64)
    bound = (d * 2.0 ** -23) * (np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64)))
    assert (np.abs(Y - want) <= bound).all()
    assert (np.abs(host(R) - want[:5000]) <= bound[:5000]).all()
