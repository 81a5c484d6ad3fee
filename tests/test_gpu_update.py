"""STEP 3's sort and chunked sums at the edges of their splits: chunks of 64 to 512 members (by the number of rows),
the scan's 32 clusters per workgroup and 1024 per round, tables past the LDS cursors, rows that belong nowhere."""
import numpy as np
import pytest

from gpu_util import host, to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return torch_cuda()


@pytest.fixture(scope="module")
def km(torch):
    import paper_2608_14648_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("n,k,d", [(1, 1, 4), (64, 1, 8), (65, 1, 8), (255, 31, 4), (257, 32, 260), (5000, 33, 4),
                                   (20000, 1025, 8), (20000, 16385, 4), (131072, 7, 64), (262145, 100, 4),
                                   (300000, 3, 1028)])
def test_f32_means_and_counts(km, torch, n, k, d):
    g = np.random.default_rng(n + k)
    X = g.standard_normal((n, d)).astype(np.float32)
    a = g.integers(0, k, n).astype(np.int32)
    if n > 100:
        a[::97] = 0             # one large cluster,
        a[5::101] = -1          # rows of no cluster,
        a[7::103] = 2 ** 31 - 1
    if k > 2:
        a[a == 2] = 1           # and an empty one
    C0 = g.standard_normal((k, d)).astype(np.float32)
    C, cnt = km.kmeans_update(km.points_f32(to_dev(X, torch)), to_dev(a, torch), to_dev(C0, torch),
                              policy=km.KM_EMPTY_KEEP)
    ok = (a >= 0) & (a < k)
    want_n = np.bincount(a[ok], minlength=k)
    np.testing.assert_array_equal(host(cnt), want_n)
    S, A = np.zeros((k, d)), np.zeros((k, d))
    np.add.at(S, a[ok], X[ok].astype(np.float64))
    np.add.at(A, a[ok], np.abs(X[ok]).astype(np.float64))
    has = want_n > 0
    C = host(C)
    np.testing.assert_array_equal(C[~has], C0[~has])
    # a value passes at most 128 + 3 fp32 additions of a wave and its chunk, then fp64, then one rounding
    bound = (132 * 2.0 ** -24 * A + 2.0 ** -24 * np.abs(S))[has] / want_n[has, None]
    assert (np.abs(C[has] - S[has] / want_n[has, None]) <= bound + 1e-30).all()


@pytest.mark.parametrize("n,k", [(1, 1), (65, 3), (5000, 33), (70000, 1300)])
def test_sq8_means_are_exact(km, torch, n, k):
    g = np.random.default_rng(n)
    d = 32
    Q = g.integers(0, 256, (n, d)).astype(np.uint8)
    a = g.integers(0, k, n).astype(np.int32)
    C, cnt = km.kmeans_update(km.points_sq8(to_dev(Q, torch)), to_dev(a, torch),
                              torch.zeros((k, d), dtype=torch.uint8, device="cuda"), policy=km.KM_EMPTY_KEEP)
    N = np.bincount(a, minlength=k)
    S = np.zeros((k, d), np.int64)
    np.add.at(S, a, Q.astype(np.int64))
    np.testing.assert_array_equal(host(cnt), N)
    has = N > 0
    np.testing.assert_array_equal(host(C)[has], ((2 * S + N[:, None]) // np.maximum(2 * N[:, None], 1))[has])


@pytest.mark.parametrize("n,k", [(9000, 1), (9000, 2), (700, 1), (40000, 3)])
@pytest.mark.parametrize("fmt", ["sign1", "lvq4"])
def test_means_of_many_chunks(km, torch, fmt, n, k):
    """Clusters of 11 to 105 chunks, which are added up eight at a time and the rest, against 64-bit means of the decoded
    points.  A chunk's alphas are multiples of its largest over 2^23 - 1, LVQ4's scales of its largest over 2^19 - 1."""
    g = np.random.default_rng(n + k)
    d = 64
    X = g.standard_normal((n, d)).astype(np.float32)
    a = g.integers(0, k, n).astype(np.int32)
    if fmt == "sign1":
        bits, m, alpha, _ = km.quantize_sign1(to_dev(X, torch))
        P = km.points_sign1(bits, alpha, m, d)
        b = (host(bits).view(np.uint32)[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1
        al = host(alpha).astype(np.float64)
        dec = host(m).astype(np.float64) + al[:, None] * (2.0 * b.reshape(n, d) - 1)
        room = 2.0 ** -23 * al.max() + 2.0 ** -22 * np.abs(dec).max()
    else:
        codes, par = km.quantize_lvq4(to_dev(X, torch))
        P = km.points_lvq4(codes, par, d)
        c = host(codes)
        c = np.stack([c & 15, c >> 4], 2).reshape(n, d).astype(np.float64)
        s, lo = host(par)[:, :1].astype(np.float64), host(par)[:, 1:2].astype(np.float64)
        dec = s * c + lo
        room = 15 * 2.0 ** -19 * s.max() + 2.0 ** -22 * np.abs(dec).max()
    C, _ = km.kmeans_update(P, to_dev(a, torch), torch.zeros((k, d), device="cuda"), policy=km.KM_EMPTY_KEEP)
    want = np.stack([dec[a == j].mean(0) for j in range(k)])
    assert (np.abs(host(C) - want) <= room).all(), np.abs(host(C) - want).max() / room
