"""What is measured: the work that programs have this library do, through its
public entry points (the HMatrix and Server classes of the binding), from the
smallest calls to the largest.

A case names the geometry (sphere surface or dielectric cube, points at 1,536
per 4 pi square wavelengths or 4,096 per cubic wavelength), the build options
that go with it, and one call:

  series   x_K, the truncated power series
  apply    y = Z_l x, one H-matvec
  gmres    x* by GMRES with the series (K = 0: D^{-1}) as preconditioner
  nested   the nested multi-level form
  refine   a fixed number of refinement passes (what a captured graph replays)
  served   requests of mixed geometries and widths through a Server
  cold     the build of a new geometry from host points, one solve, the release

`prepare` builds the handle and makes the right-hand sides (plane waves), all
from the seed; `exact` evaluates the same quantity from the uncompressed
matrix entries in FP64 (so its distance to a result is the ACA tolerance).
"""
import math
import types

import numpy as np
import torch

WAVENUMBER = 2.0 * math.pi
SURFACE, VOLUME = 0, 1


# ------------------------------------------------------------------- the cases
def _case(name, kind, n, op, nrhs=1, K=4, level=-1, f32=False, count=1, passes=0):
    """n: points (sphere) or cells per side (cube); count > 1: a batched handle
    of spheres of uneven size, the largest n; count for served: requests."""
    return {"name": name, "kind": kind, "n": n, "op": op, "nrhs": nrhs, "K": K, "level": level,
            "f32": f32, "count": count, "passes": passes}


def listed():
    return [
        # the smallest call: one plane wave on a small sphere, latency and launches
        _case("sphere_1536_series", "sphere", 1536, "series"),
        # the headline workload: one right-hand side, K = 4, leaf level, FP64
        _case("sphere_24576_series", "sphere", 24576, "series"),
        # the H-matvec with every far block, as an outer iterative solver calls it
        _case("sphere_24576_matvec", "sphere", 24576, "apply", level=0),
        # one right-hand side solved to x*: FP64 GMRES, FP32-block series inside
        _case("sphere_24576_gmres_f32", "sphere", 24576, "gmres", f32=True),
        # the paper's nested form over the leaf level and the one above it
        _case("sphere_24576_nested", "sphere", 24576, "nested", level=7),
        # many incidence angles on a volume, FP64 matrix cores
        _case("cube_32768_64rhs", "cube", 32, "series", nrhs=64, K=5),
        # the same on FP32 blocks (the result has FP32 accuracy and is kept so)
        _case("cube_32768_64rhs_f32", "cube", 32, "series", nrhs=64, K=5, f32=True),
        # an odd size with a few right-hand sides (streaming kernels)
        _case("cube_4913_7rhs", "cube", 17, "series", nrhs=7, K=5),
        # uneven spheres solved together to x*, FP32 blocks, 16 angles each
        _case("batch_64_refine_f32", "sphere", 8192, "refine", nrhs=16, f32=True, count=64, passes=49),
        # a small batch, series only, FP64
        _case("batch_16_series", "sphere", 8192, "series", nrhs=16, count=16),
        # resident geometries, requests of 1 to 64 right-hand sides solved to x*
        _case("served_mix", "mixed", 6000, "served", nrhs=64, f32=True, count=8),
        # a geometry seen for the first time: build, one solve, release
        _case("cold_sphere_5800", "sphere", 5800, "cold", nrhs=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["series", "series", "series", "apply", "gmres", "nested", "refine", "batch",
                     "served", "cold"])
    f32 = rng.random() < 0.4
    kind = "cube" if rng.random() < 0.4 else "sphere"
    n = _log(rng, 8, 32) if kind == "cube" else _log(rng, 600, 24576)
    nrhs = rng.choice([1, 1, rng.randint(2, 7), rng.randint(8, 33), rng.randint(34, 64)])
    K = rng.randint(2, 5)
    if op in ("series", "apply"):
        level = rng.choice([-1, -1, 0]) if op == "series" else rng.choice([-1, 0])
        return _case("", kind, n, op, nrhs, K, level, f32)
    if op == "gmres":
        if kind == "cube":
            return _case("", kind, min(n, 20), op, rng.randint(1, 40), 0, -1, False)
        return _case("", kind, n, op, min(nrhs, 16), K, -1, f32)
    if op == "nested":
        return _case("", "sphere", max(n, 1500) if kind == "sphere" else 300 * n, op, min(nrhs, 12),
                     rng.randint(2, 3), -2, False)
    if op == "refine":
        return _case("", "sphere", min(n, 8192) if kind == "sphere" else 250 * n, op, min(nrhs, 16), K,
                     -1, True, 1, rng.randint(20, 40))
    if op == "batch":
        return _case("", "sphere", _log(rng, 2000, 8192), "series", rng.randint(1, 32), K, -1, f32,
                     rng.randint(3, 40))
    if op == "served":
        return _case("", "mixed", _log(rng, 1500, 6000), op, rng.randint(8, 64), 4, -1, True,
                     rng.randint(3, 8))
    return _case("", "sphere", _log(rng, 600, 8192), "cold", rng.randint(1, 16), K)


# ------------------------------------------------------------------ geometries
def _problem(kind, n, rng):
    if kind == "sphere":
        a = math.sqrt(n / 1536.0)
        i = np.arange(n, dtype=np.float64)
        z = 1.0 - (2.0 * i + 1.0) / n
        r = np.sqrt(np.maximum(0.0, 1.0 - z * z))
        phi = i * (math.pi * (3.0 - math.sqrt(5.0)))
        p = np.stack([r * np.cos(phi), r * np.sin(phi), z], axis=1) * a
        p += rng.uniform(-0.01, 0.01, size=p.shape)
        p *= (a / np.linalg.norm(p, axis=1))[:, None]
        return types.SimpleNamespace(kind=SURFACE, xyz=np.ascontiguousarray(p), k=WAVENUMBER,
                                     h=math.sqrt(4.0 * math.pi * a * a / n), chi=None, n=n)
    c = (np.arange(n, dtype=np.float64) + 0.5) / 16.0
    zz, yy, xx = np.meshgrid(c, c, c, indexing="ij")
    p = np.stack([xx.ravel(), yy.ravel(), zz.ravel()], axis=1)
    p = np.ascontiguousarray(p + rng.uniform(-0.01, 0.01, size=p.shape))
    return types.SimpleNamespace(kind=VOLUME, xyz=p, k=WAVENUMBER, h=1.0 / 16.0,
                                 chi=rng.uniform(0.5, 2.0, size=n ** 3), n=n ** 3)


def _build_opts(kind, n):
    """Leaf size and ACA tolerance that go with a geometry of n points."""
    if kind == "cube":
        return 128, 1e-5
    return (64 if n <= 8192 else 128), 1e-4


def _sizes(case):
    """Sizes of a batch: log-uniform over a factor of 16, the largest first."""
    r = np.random.RandomState(case["count"])
    s = case["n"] * np.exp(-r.uniform(0.0, math.log(16.0), size=case["count"]))
    s[0] = case["n"]
    return [int(round(v)) for v in s]


def _problems(case, seed):
    rng = np.random.RandomState(seed)
    if case["op"] == "served":  # two spheres and two cubes
        side = max(8, int(round((case["n"] / 2) ** (1.0 / 3.0))))
        return [_problem("sphere", case["n"], rng), _problem("cube", side, rng),
                _problem("sphere", case["n"] // 3 + 1, rng), _problem("cube", side - 3, rng)], rng
    if case["count"] > 1:
        return [_problem("sphere", n, rng) for n in _sizes(case)], rng
    return [_problem(case["kind"], case["n"], rng)], rng


def _plane_waves(prob, nrhs, rng):
    """(n, nrhs) complex128, column-major, on the GPU."""
    d = rng.normal(size=(nrhs, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    ph = torch.from_numpy(d).cuda() @ torch.from_numpy(prob.xyz).cuda().t()
    return torch.polar(torch.ones_like(ph), -prob.k * ph).t()


def _rhs(case, probs, rng):
    b = torch.cat([_plane_waves(p, case["nrhs"], rng).t() for p in probs], dim=1)
    return b.contiguous().t() if case["nrhs"] > 1 else b.reshape(-1)


def _requests(case, probs, rng):
    """(geometry, right-hand sides) of each request, on the host."""
    widths = [1 + (i * case["nrhs"]) // max(1, case["count"] - 1) for i in range(case["count"])]
    return [(i % len(probs), np.asfortranarray(
        _plane_waves(probs[i % len(probs)], min(64, w), rng).cpu().numpy()))
        for i, w in enumerate(widths)]


def _level(case, leaf_level):
    """-2 and below count up from the leaf level."""
    return case["level"] if case["level"] >= -1 else leaf_level + 1 + case["level"]


# ------------------------------------------------------------------------ runs
def prepare(case, seed):
    from paper_2307_03968_amd import hmps
    probs, rng = _problems(case, seed)
    st = types.SimpleNamespace(case=case, hmps=hmps, probs=probs)
    st.precision = hmps.HM_F32_APPLY if case["f32"] else hmps.HM_F64
    if case["op"] == "served":
        st.server = hmps.Server(slots=2)
        st.requests = _requests(case, probs, rng)
        # every geometry resident before the stream starts
        widest = [np.asfortranarray(_plane_waves(p, 64, rng).cpu().numpy()) for p in probs]
        for t in [_submit(st, g, b, True) for g, b in enumerate(widest)]:
            st.server.wait(t)
        return st
    leaf, tol = _build_opts(case["kind"], max(p.n for p in probs))
    st.build = dict(leaf_max=leaf, aca_tol=tol)
    st.b = _rhs(case, probs, rng)
    if case["op"] == "cold":
        return st
    # a handle for many right-hand sides keeps no half-storage data
    flags = hmps.HM_BUILD_NO_HALF if case["count"] > 1 else 0
    st.h = hmps.HMatrix(probs if case["count"] > 1 else probs[0], flags=flags, **st.build)
    st.level = _level(case, st.h.info()["leaf_level"])
    return st


def _submit(st, g, b, first=False):
    p, case = st.probs[g], st.case
    surface = p.kind == SURFACE
    leaf, tol = _build_opts("sphere" if surface else "cube", p.n)
    return st.server.submit(
        g, b, K=case["K"] if surface else 0, kind=st.hmps.PS_GMRES, max_passes=500, refine_tol=1e-10,
        precision=st.precision if surface else st.hmps.HM_F64, prob=p if first else None,
        leaf_max=leaf, aca_tol=tol, restart=20)


def run(st):
    case, hmps = st.case, st.hmps
    if case["op"] == "served":
        return [st.server.wait(t)[0] for t in [_submit(st, g, b) for g, b in st.requests]]
    if case["op"] == "cold":
        h = hmps.HMatrix(st.probs[0], **st.build)
        x = h.solve(st.b, K=case["K"], precision=st.precision)
        h.close()
        return x
    if case["op"] == "apply":
        y = st.h.apply(st.b, level=st.level, precision=st.precision)
    elif case["op"] == "gmres":
        return st.h.solve(st.b, K=case["K"], level=st.level, precision=st.precision,
                          kind=hmps.PS_GMRES, max_passes=500, refine_tol=1e-10)
    elif case["op"] == "refine":
        return st.h.solve(st.b, K=case["K"], level=st.level, precision=st.precision,
                          kind=hmps.PS_REFINE_FIXED, max_passes=case["passes"])
    else:
        kind = hmps.PS_NESTED if case["op"] == "nested" else hmps.PS_SERIES
        y = st.h.solve(st.b, K=case["K"], level=st.level, precision=st.precision, kind=kind)
    # products of FP32 blocks without refinement are FP32 results
    return y.to(torch.complex64) if case["f32"] else y


# ----------------------------------------------- tree and partition (plain numpy)
def _tree(xyz, leaf_max):
    """Median bisection of the longest bounding-box axis: perm and node arrays
    (offset, size, depth, first child or -1, bounding box)."""
    perm = np.arange(xyz.shape[0])
    nodes, boxes, todo = [[0, xyz.shape[0], 0, -1]], [None], [0]
    while todo:
        i = todo.pop()
        off, size, depth, _ = nodes[i]
        pts = xyz[perm[off:off + size]]
        lo, hi = pts.min(axis=0), pts.max(axis=0)
        boxes[i] = (lo, hi)
        if size <= leaf_max:
            continue
        ax = int(np.argmax(hi - lo))
        idx = perm[off:off + size]
        perm[off:off + size] = idx[np.lexsort((idx, pts[:, ax]))]
        half = size // 2
        nodes[i][3] = len(nodes)
        nodes += [[off, half, depth + 1, -1], [off + half, size - half, depth + 1, -1]]
        boxes += [None, None]
        todo += [len(nodes) - 2, len(nodes) - 1]
    nd = np.array(nodes)
    return perm, nd, np.array([b[0] for b in boxes]), np.array([b[1] for b in boxes])


def _partition(nd, lo, hi):
    """(near pairs, far pairs) of node ids by the admissibility
    min(diam) <= dist of the bounding boxes."""
    diam = np.sqrt(((hi - lo) ** 2).sum(axis=1))
    near, far = [], []
    t, s = np.zeros(1, int), np.zeros(1, int)
    while t.size:
        gap = np.maximum(0.0, np.maximum(lo[s] - hi[t], lo[t] - hi[s]))
        adm = (t != s) & (np.sqrt((gap ** 2).sum(axis=1)) >= np.minimum(diam[t], diam[s]))
        tl, sl = nd[t, 3] < 0, nd[s, 3] < 0
        both = ~adm & tl & sl
        far.append(np.stack([t[adm], s[adm]], 1))
        near.append(np.stack([t[both], s[both]], 1))
        go = ~adm & ~both
        t, s, tl, sl = t[go], s[go], tl[go], sl[go]
        nt, ns = [], []
        for a in (0, 1):
            for b in (0, 1):
                ok = ~(tl & (a == 1)) & ~(sl & (b == 1))
                nt.append(np.where(tl, t, nd[t, 3] + a)[ok])
                ns.append(np.where(sl, s, nd[s, 3] + b)[ok])
        t, s = np.concatenate(nt), np.concatenate(ns)
    return np.concatenate(near), np.concatenate(far)


# ------------------------------------------------------------------------ work
def _entries(kind, n):
    """(diagonal, near t < s, far factor entries by distance above the leaf
    level) that determine the operator: it is symmetric up to a diagonal
    scaling, so each off-diagonal block counts once.  Ranks are the mean ones
    of the tolerance (4 at 1e-4 on a surface, 9 at 1e-5 in a volume)."""
    prob = _problem(kind, n, np.random.RandomState(0))
    perm, nd, lo, hi = _tree(prob.xyz, _build_opts(kind, prob.n)[0])
    near, far = _partition(nd, lo, hi)
    sz, L = nd[:, 1], int(nd[:, 2].max())
    pairs = sz[near[:, 0]] * sz[near[:, 1]]
    diag = int(pairs[near[:, 0] == near[:, 1]].sum())
    level = np.maximum(nd[far[:, 0], 2], nd[far[:, 1], 2])
    ent = (4 if kind == "sphere" else 9) * (sz[far[:, 0]] + sz[far[:, 1]])
    up = {int(L - l): int(ent[level == l].sum()) // 2 for l in np.unique(level)}
    return diag, (int(pairs.sum()) - diag) // 2, up


def work(case):
    """Operator entries once per product (the products of a series depend on
    each other and the operator exceeds the caches; below 256 MB it counts
    once), vectors read and written once."""
    if case["op"] == "served":
        side = max(8, int(round((case["n"] / 2) ** (1.0 / 3.0))))
        geoms = [("sphere", case["n"]), ("cube", side), ("sphere", case["n"] // 3 + 1),
                 ("cube", side - 3)]
    else:
        kind = "sphere" if case["count"] > 1 else case["kind"]
        geoms = [(kind, n) for n in (_sizes(case) if case["count"] > 1 else [case["n"]])]
    K, total = case["K"], {"bytes": 0.0, "flops": 0.0}
    for kind, n in geoms:
        diag, near, up = _entries(kind, n)
        pts = n if kind == "sphere" else n ** 3
        nrhs = case["nrhs"]
        deepest = {-1: 0, 0: 99}.get(case["level"], 1)
        term = near + sum(e for d, e in up.items() if d <= deepest)
        products = {"series": K, "apply": 1, "cold": K, "gmres": 25 * (K + 1), "served": 25 * (K + 1),
                    "refine": (case["passes"] + 1) * (K + 1), "nested": K}[case["op"]]
        if case["op"] == "nested":  # K outer products with the coarser factor, K more inside each
            coarse = sum(e for d, e in up.items() if 0 < d <= deepest)
            ent = K * (K + 2) * (near + up.get(0, 0)) + K * coarse
        else:
            ent = products * term
        size = (8 if case["f32"] else 16) * (term + diag)
        moved = (8 if case["f32"] else 16) * ent if size > 256e6 else size
        if case["op"] == "cold":
            moved = 16 * (term + diag)
        total["bytes"] += moved + 16 * 2 * pts * nrhs
        total["flops"] += 8.0 * 2 * ent * nrhs
    return total


# ----------------------------------------------------------------------- exact
class _Dense:
    """The matrices of one geometry from its entries, tree order, on the GPU."""

    def __init__(self, prob, kind):
        self.perm, nd, lo, hi = _tree(prob.xyz, _build_opts(kind, prob.n)[0])
        near, far = _partition(nd, lo, hi)
        leaves = np.array(sorted(np.flatnonzero(nd[:, 3] < 0), key=lambda i: nd[i, 0]))
        self.off, self.size, self.L = nd[leaves, 0], nd[leaves, 1], int(nd[:, 2].max())
        nl, n = len(leaves), prob.n
        leaf_of = np.repeat(np.arange(nl), self.size)
        # level of the far block that covers a pair of leaves; near blocks 98, diagonal 99
        lev = np.full((nl, nl), -1, dtype=np.int64)
        first, last = leaf_of[nd[:, 0]], leaf_of[nd[:, 0] + nd[:, 1] - 1]
        for t, s in far:
            lev[first[t]:last[t] + 1, first[s]:last[s] + 1] = max(nd[t, 2], nd[s, 2])
        for t, s in near:
            lev[first[t], first[s]] = 99 if t == s else 98
        self.lev = torch.from_numpy(lev).cuda()
        self.leaf_of = torch.from_numpy(leaf_of).cuda()
        self.x = torch.from_numpy(prob.xyz[self.perm]).cuda()
        self.chi = None if prob.chi is None else torch.from_numpy(prob.chi[self.perm]).cuda()
        self.prob, self.n = prob, n
        self.Dinv = None

    def matrix(self, lo, hi):
        """Z restricted to the blocks whose level lies in [lo, hi]."""
        p, n = self.prob, self.n
        out = torch.empty(n, n, dtype=torch.complex128, device="cuda")
        scale = (p.h ** 2 if p.kind == SURFACE else p.k ** 2 * p.h ** 3) / (4.0 * math.pi)
        for r in range(0, n, 1024):
            e = min(n, r + 1024)
            d = (self.x[r:e, None, :] - self.x[None, :, :]).square().sum(-1).sqrt()
            row = torch.arange(r, e, device="cuda")
            d[row - r, row] = 1.0
            z = torch.polar(scale / d, -p.k * d)
            if p.kind == VOLUME:
                z *= self.chi[None, :]
                z[row - r, row] = (1.0 / self.chi[r:e] + 0.5).to(z.dtype)
            else:
                z[row - r, row] = complex(2.0 * p.h, 0.2 * p.h)
            lv = self.lev[self.leaf_of[r:e]][:, self.leaf_of]
            out[r:e] = torch.where((lv >= lo) & (lv <= hi), z, torch.zeros_like(z))
        return out

    def dinv(self, v):
        """D^{-1} v."""
        if self.Dinv is None:
            Z = self.matrix(99, 99)
            self.Dinv = [torch.linalg.inv(Z[o:o + m, o:o + m]) for o, m in zip(self.off, self.size)]
        return torch.cat([D @ v[o:o + m] for D, o, m in zip(self.Dinv, self.off, self.size)])

    def series(self, R, v, terms):
        """sum_{k <= terms} (-D^{-1} R)^k D^{-1} v."""
        x = y = self.dinv(v)
        for _ in range(terms):
            y = -self.dinv(R @ y)
            x = x + y
        return x


def _exact_one(case, prob, kind, b):
    M = _Dense(prob, kind)
    v = b.reshape(prob.n, -1)[torch.from_numpy(M.perm).cuda()]
    op, K = case["op"], case["K"]
    level = _level(case, M.L)
    level = M.L if level < 0 else level
    if op == "apply":
        x = M.matrix(level, 99) @ v
    elif op == "nested":
        R = [M.matrix(M.L, 98)] + [M.matrix(l, l) for l in range(M.L - 1, level - 1, -1)
                                   if bool((M.lev == l).any())]

        def inverses(j, u):  # the first j truncated inverses
            for i in range(j):
                y = u
                for _ in range(K):
                    y = -inverses(i, M.dinv(R[i] @ y))
                    u = u + y
            return u

        x = inverses(len(R), M.dinv(v))
    elif op in ("gmres", "served"):
        if prob.n > 14000:  # the series converges on a sphere: summed to rounding
            x = M.series(M.matrix(level, 98), v, 600)
        else:
            x = torch.linalg.solve(M.matrix(level, 99), v)
    else:
        terms = (K + 1) * (case["passes"] + 1) - 1 if op == "refine" else K
        x = M.series(M.matrix(level, 98), v, terms)
    out = torch.empty_like(x)
    out[torch.from_numpy(M.perm).cuda()] = x
    return out


def exact(case, seed):
    probs, rng = _problems(case, seed)
    kinds = ["sphere" if p.kind == SURFACE else "cube" for p in probs]
    if case["op"] == "served":
        return [_exact_one(case, probs[g], kinds[g], torch.from_numpy(b).cuda())
                for g, b in _requests(case, probs, rng)]
    b = _rhs(case, probs, rng)
    big = max(p.n for p in probs)  # the leaf size of a batch follows its largest instance
    parts, at = [], 0
    for p, k in zip(probs, kinds):
        if _build_opts(k, p.n) != _build_opts(k, big):
            return None
        parts.append(_exact_one(case, p, k, b[at:at + p.n]))
        at += p.n
    x = torch.cat(parts)
    return x.reshape(-1) if case["nrhs"] == 1 else x
