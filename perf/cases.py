"""The calls this framework's speed is judged by: whole passes through the public entry points.

`listed()` names twelve calls a user of the library makes, over the range of sizes, point formats and options;
`draw()` gives more of the same ranges.  `prepare()` makes what the user's program holds before the call (vectors
in HBM drawn from the Gaussian-mixture recipe of `synth`, start rows, a basis or rotation), `run()` is one pass,
`exact()` the same outputs in 64 bits by plain torch where they have such a value.

The kinds of pass:
  assign  STEP 2 for given centroids (building an index's lists, serving a batch of queries)
  fit     encode the vectors in the format, then Lloyd for T iterations (the index build)
  update  STEP 3 for a given assignment
  encode  the encoding of the vectors alone
  pca     covariance of the vectors and their projection on a given basis
  fine    Lloyd inside given meso-clusters (the second level of a hierarchical build)
  hier    the whole two-level build
  pruned  one pruned STEP 2 from the previous assignment
"""
import math

import torch

import paper_2608_14648_amd as km

DEV = "cuda"
ROWS = 1 << 16  # rows generated or checked at a time


# ---- the cases ---------------------------------------------------------------------------------------------------

def listed():
    return [
        # a batch of queries against the coarse centroids of a served index, into buffers the server keeps: latency
        dict(name="assign_f32_1k_d768_k1000", kind="assign", fmt="f32", n=1024, d=768, k=1000, noalloc=True),
        # the smallest index build of the benchmark: launches count
        dict(name="fit_f32_20k_d128_k64", kind="fit", fmt="f32", n=20_000, d=128, k=64, iters=10),
        # raw vectors of a middling collection (the shape of arXiv / Jina embeddings)
        dict(name="fit_f32_1m_d768_k1000", kind="fit", fmt="f32", n=1_000_000, d=768, k=1000, iters=4),
        # the flagship: ten million vectors after PCA to 256 dims, one pass of STEP 2
        dict(name="assign_f32_10m_d256_k4096", kind="assign", fmt="f32", n=10_000_000, d=256, k=4096, noalloc=False),
        # the same collection as 8-bit codes, encode included
        dict(name="fit_sq8_1m_d768_k1000", kind="fit", fmt="sq8", n=1_000_000, d=768, k=1000, iters=10),
        # 1-bit codes around the mean (the shape of MXBAI embeddings), encode included
        dict(name="fit_sign1_1m_d1024_k1024", kind="fit", fmt="sign1", n=1_000_000, d=1024, k=1024, iters=10),
        # 4-bit codes at a ragged size
        dict(name="fit_lvq4_250k_d416_k601", kind="fit", fmt="lvq4", n=250_007, d=416, k=601, iters=10),
        # RabitQ as the paper runs it: rotation, codes, Lloyd, the last update from the rotated rows
        dict(name="fit_rabitq_500k_d1024_k1024", kind="fit", fmt="rabitq", n=500_000, d=1024, k=1024, iters=6),
        # an exact front segment plus 1-bit tail, one pass of STEP 2 with its objective
        dict(name="assign_hybrid_2m_d1024_k4096", kind="assign", fmt="hybrid", n=2_000_000, d=1024, k=4096,
             d_front=384, noalloc=False),
        # PCA of 1024-dim vectors to 256 dims
        dict(name="pca_2m_d1024_to256", kind="pca", n=2_000_000, d=1024, d_out=256),
        # the fine level of a hierarchical build: about 63 meso-clusters of uneven size, 4000 fine clusters (started
        # from the points inside, so one iteration: after that its near ties lead two right answers apart)
        dict(name="fine_f32_1m_d1024_k4000", kind="fine", fmt="f32", n=1_000_000, d=1024, k=4000, iters=1),
        # a settled pass of Lloyd with dimension pruning
        dict(name="pruned_f32_1m_d768_k1000", kind="pruned", fmt="f32", n=1_000_000, d=768, k=1000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["assign", "assign", "assign", "fit", "fit", "fit", "fit", "update", "update", "encode", "pca",
                       "fine", "hier", "pruned"])
    if kind in ("hier",):
        fmt = "sq8"
    elif kind in ("fine", "pruned"):
        fmt = rng.choice(["f32", "sq8"])
    elif kind == "encode":
        fmt = rng.choice(["sq8", "sign1", "rabitq", "lvq4", "bf16"])
    else:
        fmt = rng.choice(["f32", "f32", "f32", "sq8", "sign1", "hybrid", "rabitq", "lvq4", "bf16"])
    unit = {"f32": 4, "bf16": 8, "sq8": 16}.get(fmt, 32)
    d = unit * max(1, _log(rng, 64, 1536) // unit)
    if kind == "pca":
        d = 4 * (_log(rng, 128, 1536) // 4)
        n = _log(rng, 2_000, 1_000_000)
        return dict(kind=kind, n=n, d=d, d_out=4 * max(1, rng.randint(d // 8, d // 2) // 4))
    if kind in ("hier", "fine"):
        n = _log(rng, 50_000, 1_000_000)
        k = int(4 * math.sqrt(n))
        c = dict(kind=kind, fmt=fmt, n=n, d=d, k=k, iters=rng.randint(2, 5) if kind == "hier" else 1)
    elif kind == "encode":
        return dict(kind=kind, fmt=fmt, n=_log(rng, 1_000, 1_000_000), d=d)
    elif kind == "pruned":
        d = 16 * max(8, d // 16)
        return dict(kind=kind, fmt=fmt, n=_log(rng, 20_000, 1_000_000), d=d, k=_log(rng, 64, 2048))
    else:
        n = _log(rng, 1_000, 2_000_000)
        k = max(2, min(_log(rng, 16, 4096), n // 8))
        c = dict(kind=kind, fmt=fmt, n=n, d=d, k=k)
        if kind == "fit":
            c["iters"] = rng.randint(2, 10)
        if kind == "assign":
            c["noalloc"] = n <= 100_000 and rng.random() < 0.5
    if fmt == "hybrid":
        c["d"] = d = max(64, d)
        c["d_front"] = 32 * max(1, (d * 3 // 8) // 32)
    # no dearer than the largest listed call
    most = 1.0e13 / (1 if fmt in ("f32", "hybrid", "bf16") else 0.25)
    c["n"] = max(1000, min(c["n"], int(most / (c["k"] * d * (c.get("iters", 0) + 1))), int(1.5e9 / d)))
    if "noalloc" in c:
        c["noalloc"] = c["noalloc"] and c["n"] <= 100_000
    return c


# ---- inputs ------------------------------------------------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1009 + salt)
    return g


def _mixture(n, d, comps, seed, sigma=0.15, normalize=True, power=0.0):
    """Rows of a Gaussian mixture in random order (unit norm if `normalize`), and one row of every component: the
    start a careful seeding finds.  From random rows several centroids share a component and others have none, and
    Lloyd then follows its near ties: two right answers soon differ."""
    g = _gen(seed, 1)
    scale = torch.arange(1, d + 1, device=DEV, dtype=torch.float32).pow(-0.5 * power)
    means = torch.randn(comps, d, generator=g, device=DEV) * scale
    order = torch.randperm(n, generator=g, device=DEV)
    X = torch.empty(n, d, device=DEV)
    for lo in range(0, n, ROWS):
        x = X[lo:lo + ROWS]
        x.normal_(generator=g)
        x.mul_(sigma * scale)
        x.add_(means[order[lo:lo + ROWS] % comps])
        if normalize:
            x.div_(x.norm(dim=1, keepdim=True))
    return X, order.argsort()[:comps]


def _vectors(case, seed):
    n, d = case["n"], case["d"]
    k = case.get("k", 256)
    if case["kind"] == "fit" and n <= 50_000:  # the smoke-size recipe: wide components, not normalised
        return _mixture(n, d, k, seed, sigma=0.3, normalize=False)
    decays = case["kind"] in ("pca", "fine", "hier") or case.get("fmt") == "hybrid" or k >= 4000
    return _mixture(n, d, k, seed, power=0.5 if decays else 0.0)


def _orthogonal(d, cols, seed):
    q, _ = torch.linalg.qr(torch.randn(d, d, generator=_gen(seed, 3), device=DEV, dtype=torch.float64))
    return q[:, :cols].float().contiguous()


def _encode(fmt, X, s):
    """The encoder's outputs and the points made of them, as a program builds them from its vectors."""
    if fmt == "f32":
        return [], km.points_f32(X)
    if fmt == "bf16":
        Xb = km.quantize_bf16(X)
        return [Xb], km.points_bf16(Xb)
    if fmt == "sq8":
        codes, params = km.quantize_sq8(X)
        return [codes, params], km.points_sq8(codes)
    if fmt == "lvq4":
        codes, par = km.quantize_lvq4(X)
        return [codes, par], km.points_lvq4(codes, par, X.shape[1])
    if fmt == "rabitq":
        bits, m, alpha, Y = km.rabitq_encode(X, s["rotation"], want_rotated=True)
        return [bits, m, alpha, Y], km.points_rabitq(bits, alpha, X.shape[1], raw=Y)
    if fmt == "sign1":
        bits, m, alpha, _ = km.quantize_sign1(X)
        return [bits, m, alpha], km.points_sign1(bits, alpha, m, X.shape[1])
    df = s["d_front"]
    bits, m, alpha, front = km.quantize_sign1(X, d_front=df, want_front=True)
    return [bits, m, alpha, front], km.points_hybrid(front, bits, alpha, m, X.shape[1])


def _nearest(X, C):
    """Nearest row of C for every row of X in single precision (the previous pass's assignment)."""
    cn = (C * C).sum(1)
    out = torch.empty(X.shape[0], dtype=torch.int32, device=DEV)
    for lo in range(0, X.shape[0], ROWS):
        out[lo:lo + ROWS] = (cn - 2 * (X[lo:lo + ROWS] @ C.T)).argmin(1).int()
    return out


def _means(X, a, C):
    """The mean of every cluster's rows; an empty cluster keeps its row of C."""
    S = torch.zeros(C.shape, device=DEV, dtype=torch.float64)
    for lo in range(0, X.shape[0], ROWS):
        S.index_add_(0, a[lo:lo + ROWS].long(), X[lo:lo + ROWS].double())
    cnt = torch.bincount(a.long(), minlength=C.shape[0])
    return torch.where(cnt[:, None] > 0, S / cnt.clamp(min=1)[:, None], C.double()), cnt


def prepare(case, seed):
    kind, fmt, n, d = case["kind"], case.get("fmt"), case["n"], case["d"]
    s = dict(case)
    X, start = _vectors(case, seed)
    if fmt == "rabitq":
        s["rotation"] = _orthogonal(d, d, seed)
    if kind == "pca":
        s.update(X=X, W=_orthogonal(d, case["d_out"], seed))
    elif kind in ("fit", "encode"):
        s["X"] = X
        if kind == "fit":
            s["rows"] = start.cpu().numpy()
    elif kind == "hier":
        s["X"] = X
        s["rows"] = start[:int(round(math.sqrt(case["k"])))].cpu().numpy()
    else:
        # the clustering in the middle of its work: compressed points and the centroids two iterations in
        k_start = int(round(math.sqrt(case["k"]))) if kind == "fine" else case["k"]
        rows = start[:k_start]
        C = X[rows]
        part = X[:min(n, max(20 * k_start, 50_000))]
        C = _means(part, _nearest(part, C), C)[0].float()
        _, s["P"] = _encode(fmt, X, s)
        if kind == "fine":
            s["meso"] = _nearest(X, C)
            s["k_meso"] = k_start
        elif fmt == "sq8":
            Xc = s["P"].data.float()
            s["C"] = _means(Xc, _nearest(X, C), Xc[rows])[0].round().to(torch.uint8)
            if kind == "pruned":
                s["prev"] = _nearest(Xc, s["C"].float())
        elif fmt == "rabitq":
            s["C"] = ((C - X.mean(0)) @ s["rotation"]).contiguous()
        else:
            s["C"] = C.contiguous()
        if kind == "update":
            s["a"] = _nearest(X, C)
        elif kind == "pruned" and fmt == "f32":
            s["prev"] = _nearest(X, C)
        if case.get("noalloc"):
            s["out"] = [torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV)]
    return s


# ---- one pass ----------------------------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "assign":
        if s["noalloc"]:
            return list(km.kmeans_assign_noalloc(s["P"], s["C"], *s["out"])[:2])
        return list(km.kmeans_assign(s["P"], s["C"], score=True, objective=True))
    if kind == "fit":
        out, P = _encode(s["fmt"], s["X"], s)
        return out + list(km.kmeans_fit(P, s["k"], s["iters"], s["rows"]))
    if kind == "update":
        return list(km.kmeans_update(s["P"], s["a"], s["C"], policy=km.KM_EMPTY_KEEP))
    if kind == "encode":
        return _encode(s["fmt"], s["X"], s)[0]
    if kind == "pca":
        mean, cov = km.pca_fit_cov(s["X"])
        return [mean, cov, km.pca_project(s["X"], mean, s["W"])]
    if kind == "fine":
        return list(km.kmeans_fine(s["P"], s["meso"], s["k_meso"], s["k"], s["iters"], objective=True))
    if kind == "hier":
        codes, P = _encode(s["fmt"], s["X"], s)
        return codes + list(km.kmeans_fit_hier(P, s["k"], s["rows"], s["iters"], s["iters"], meso=True)[:4])
    return list(km.kmeans_assign_pruned(s["P"], s["C"], s["prev"], objective=True)[:3])


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def _row_bytes(case):
    d = case["d"]
    return {"f32": 4 * d, "bf16": 2 * d, "sq8": d, "lvq4": d / 2 + 16, "sign1": d / 8 + 4, "rabitq": d / 8 + 4,
            "hybrid": 4 * case.get("d_front", 0) + (d - case.get("d_front", 0)) / 8 + 4}[case["fmt"]]


def work(case):
    kind, n, d = case["kind"], case["n"], case["d"]
    if kind == "pca":
        o = case["d_out"]
        return {"bytes": 4 * n * (2 * d + o) + 4 * d * (d + o), "flops": n * d * (d + 1) + 2 * n * d * o}
    row = _row_bytes(case)
    if kind == "encode":
        fits = 4 * d if case["fmt"] in ("sq8", "sign1", "rabitq") else 0  # the statistics need a pass of their own
        turns = case["fmt"] == "rabitq"
        return {"bytes": n * (4 * d + fits + row + (4 * d if turns else 0)),
                "flops": n * d * (2 * d if turns else 2)}
    k = case["k"]
    c = k * d * (1 if case["fmt"] == "sq8" else 4)
    pass_b, pass_f = n * row + c + 4 * n, 2 * n * k * d
    if kind == "assign":
        return {"bytes": pass_b + 4 * n, "flops": pass_f}
    if kind == "update":
        return {"bytes": n * row + 4 * n + c, "flops": n * d}
    if kind == "pruned":  # the front dims of every pair, then the previous centroid's distance
        df = min(d, 32 * math.ceil(d / 8 / 32))
        return {"bytes": pass_b + 12 * n, "flops": 2 * n * k * df + 3 * n * d}
    # every iteration needs the points once; the update's sums are of the rows that its assignment read
    t = case["iters"]
    enc = work(dict(case, kind="encode")) if kind in ("fit", "hier") and case["fmt"] != "f32" else \
        {"bytes": 0, "flops": 0}
    if kind == "fit":
        return {"bytes": enc["bytes"] + (t + 1) * pass_b, "flops": enc["flops"] + (t + 1) * pass_f + t * n * d}
    km_ = round(math.sqrt(k))
    fine_b, fine_f = (t + 1) * pass_b, (t + 1) * 2 * n * d * k / km_ + t * n * d
    if kind == "fine":
        return {"bytes": fine_b + 4 * n, "flops": fine_f}
    return {"bytes": enc["bytes"] + 2 * fine_b, "flops": enc["flops"] + (t + 1) * 2 * n * d * km_ + fine_f}


# ---- how far two right answers lie apart -------------------------------------------------------------------------

def tolerance(case):
    """About four times what the outputs moved by when the inputs changed in their last bit (other sums, other order)."""
    kind, fmt = case["kind"], case.get("fmt")
    if kind == "encode":
        # codes are integers in a fixed fp32 order; a rotated value next to 0 may change its sign bit
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4 if fmt == "rabitq" else 0.0}
    if kind == "pca":
        return {"rel": 1e-5, "max": 1e-3}
    if fmt == "sq8":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}  # integers throughout: nothing may differ
    if kind == "update":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    if kind == "fine":  # started from points inside the clusters: a few near ties fall the other way
        return {"rel": 1e-3, "max": 0.2, "differ": 1e-4}
    if kind == "fit" and fmt in ("bf16", "lvq4", "rabitq"):
        # centroids are rounded to 16 bits or coded in every pass, rotated points in their sign bits
        return {"rel": 1e-4, "max": 2e-2, "differ": 1e-4}
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4}


# ---- the same outputs in 64 bits ---------------------------------------------------------------------------------

def _scores(X, C, rows=1 << 14):
    """(index, ||c||^2 - 2<x, c>) of the nearest rows of C, in 64 bits."""
    C = C.double()
    cn = (C * C).sum(1)
    a = torch.empty(X.shape[0], dtype=torch.int64, device=DEV)
    sc = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
    for lo in range(0, X.shape[0], rows):
        sc[lo:lo + rows], a[lo:lo + rows] = (cn - 2 * (X[lo:lo + rows].double() @ C.T)).min(1)
    return a, sc


def _norms(X):
    return torch.cat([X[lo:lo + ROWS].double().square().sum(1) for lo in range(0, X.shape[0], ROWS)])


def _exact_hybrid(s):
    """STEP 2 on the exact front plus the 1-bit tail against int8 residual codes of the centroids."""
    P, C, df, d = s["P"], s["C"], s["d_front"], s["d"]
    r = (C - P.center)[:, df:]
    top = r.abs().amax(1)
    sigma = top / 127
    q = torch.where(top[:, None] > 0, (r / sigma[:, None]).round().clamp(-127, 127), torch.zeros_like(r)).double()
    u = sigma.double().square() * q.square().sum(1)
    Cf = C[:, :df].double()
    cn = Cf.square().sum(1)
    n = P.n
    sc = torch.empty(n, dtype=torch.float64, device=DEV)
    obj = torch.zeros((), dtype=torch.float64, device=DEV)
    bit = torch.arange(32, device=DEV, dtype=torch.int32)
    for lo in range(0, n, 1 << 14):
        w = P.data[lo:lo + (1 << 14), df // 32:]
        pm = (((w[:, :, None] >> bit) & 1) * 2 - 1).reshape(w.shape[0], -1).double()
        al = P.alpha[lo:lo + (1 << 14)].double()
        f = P.front[lo:lo + (1 << 14)].double()
        best = (cn - 2 * (f @ Cf.T) + u - 2 * al[:, None] * sigma.double() * (pm @ q.T)).amin(1)
        sc[lo:lo + (1 << 14)] = best
        obj += (best + f.square().sum(1) + al.square() * (d - df)).sum()
    return [None, sc, obj.reshape(1)]


def _exact_pruned(s):
    """The pruning test of every (point, centroid) pair on 64-bit partial distances."""
    X, C, d = s["P"].data.double() if s["n"] * s["d"] < 2e8 else s["P"].data, s["C"].double(), s["d"]
    D0 = min(d, 32 * math.ceil(d / 8 / 32))
    marks = list(range(D0, d, 64)) + [d]
    dist = torch.empty(s["n"], dtype=torch.float64, device=DEV)
    cn = torch.cumsum(C.square(), 1)
    for lo in range(0, s["n"], 1 << 14):
        x = X[lo:lo + (1 << 14)].double()
        xn = torch.cumsum(x.square(), 1)
        prev = s["prev"][lo:lo + (1 << 14)].long()[:, None]
        tau = (x - C[prev[:, 0]]).square().sum(1)
        alive = torch.ones(x.shape[0], C.shape[0], dtype=torch.bool, device=DEV)
        dot = torch.zeros(x.shape[0], C.shape[0], dtype=torch.float64, device=DEV)
        at = 0
        for D in marks:
            dot += x[:, at:D] @ C[:, at:D].T
            p = xn[:, D - 1:D] + cn[:, D - 1] - 2 * dot
            at = D
            if D < d:
                alive &= p <= (tau * ((1 + 2.1 / math.sqrt(D)) ** 2 * D / d))[:, None]
        alive.scatter_(1, prev, True)
        dist[lo:lo + (1 << 14)] = torch.where(alive, p, torch.full_like(p, math.inf)).amin(1)
    return [None, dist, dist.sum().reshape(1)]


def exact(case, seed):
    kind, fmt = case["kind"], case.get("fmt")
    if kind in ("encode", "hier", "fine"):
        # codes are whole numbers in a fixed order; a two-level build follows its near ties from level to level
        return None
    s = prepare(case, seed)
    if kind == "pca":
        X = s["X"]
        n = X.shape[0]
        mean = sum(X[lo:lo + ROWS].double().sum(0) for lo in range(0, n, ROWS)) / n
        cov = torch.zeros(case["d"], case["d"], dtype=torch.float64, device=DEV)
        Y = torch.empty(n, case["d_out"], dtype=torch.float64, device=DEV)
        for lo in range(0, n, ROWS):
            x = X[lo:lo + ROWS].double() - mean
            cov += x.T.contiguous() @ x
            Y[lo:lo + ROWS] = x @ s["W"].double()
        return [mean, cov / n, Y]
    if kind == "pruned":
        return _exact_pruned(s)
    if kind == "update":
        if fmt in ("f32", "bf16"):
            return [_means(s["P"].data, s["a"], s["C"])[0], None]
        return None
    if kind == "assign":
        n = case["n"]
        if fmt in ("f32", "bf16"):
            X = s["P"].data
            sc = _scores(X, s["C"] if fmt == "f32" else s["C"].bfloat16())[1]
        elif fmt == "sq8":
            X = torch.cat([s["P"].data[lo:lo + ROWS].float() - 128 for lo in range(0, n, ROWS)])
            sc = _scores(X, s["C"].double() - 128)[1]
        elif fmt == "hybrid":
            out = _exact_hybrid(s)
            return out[:2] if case["noalloc"] else out
        else:
            return None  # scores in a fixed fp32 order
        return [None, sc] if case["noalloc"] else [None, sc, (sc.sum() + _norms(X).sum()).reshape(1)]
    # fit: the centroids and the objective of every pass
    if fmt != "f32":
        return None
    X, C = s["X"], s["X"][torch.from_numpy(s["rows"]).to(DEV)].double()
    J, xn = [], _norms(X).sum()
    for t in range(case["iters"] + 1):
        a, sc = _scores(X, C)
        J.append(sc.sum() + xn)
        if t < case["iters"]:
            C, cnt = _means(X, a, C)
            if int(cnt.min()) == 0:  # an empty cluster splits another: not followed here
                return None
    return [C, None, torch.stack(J)]
