"""Graphs and the nested solve's level lists, which its first call outside a
capture makes: a graph captured before that call refers to the workspace, which
the call leaves where it is; and a nested solve captured before the lists exist
takes the general form."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


def _chain(depth=7, leaf=32, n=4139):
    """Clusters on a line, one tree node each at `depth`: 32 points in one spot,
    or 33 in two.  With a small eta only the spots are far from each other, the
    85 undivided ones (3,570 pairs, in fours) on the level above the leaf level;
    with the 3,655 pairs of that level pieces hold eight, so that the list of the
    one level has more partial rows than that of both."""
    sizes = []

    def halve(size, d):
        if d == depth:
            sizes.append(size)
        else:
            halve(size // 2, d + 1)
            halve(size - size // 2, d + 1)

    halve(n, 0)
    rng = np.random.default_rng(0)
    spots = [(x, c) for i, s in enumerate(sizes)
             for x, c in ([(i, s)] if s <= leaf else [(i - 0.45, s // 2), (i + 0.45, s - s // 2)])]
    xyz = np.concatenate([[x, 0.0, 0.0] + rng.uniform(-1e-5, 1e-5, (c, 3)) for x, c in spots])
    return W.Problem(W.SURFACE, xyz, W.WAVENUMBER, 1e-5)


def _capture(call):
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        call()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    return g


def test_graph_outlives_the_first_nested_call():
    prob = _chain()
    h = hmps.HMatrix(prob, 32, eta=5e-3, aca_tol=1e-4)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    lev = h.info()["leaf_level"] - 1
    assert h.info()["half_entries"][lev] > 0  # the half lists serve it
    want = h.solve(d, K=3, level=lev).cpu().numpy()
    out = torch.empty_like(d)
    g = _capture(lambda: h.solve(d, K=3, level=lev, out=out))
    x = None
    for rep in range(3):
        print(f"[gpu-case] series replay {rep}", flush=True)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want), rep
        xr = h.solve(d, K=2, level=lev, kind=hmps.PS_NESTED).cpu().numpy()  # makes the list
        x = xr if x is None else x
        assert np.array_equal(xr, x)
    h.tune(half_storage=2)  # the general form on the panels
    ref = h.solve(d, K=2, level=lev, kind=hmps.PS_NESTED).cpu().numpy()
    assert np.linalg.norm(x - ref) <= 1e-10 * np.linalg.norm(ref)
    del g
    h.close()


def test_nested_captured_before_its_lists():
    """The pool exists (from two right-hand sides), the lists do not."""
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    B = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.directions(2, 3)))).to("cuda")
    d = B[:, 0].contiguous()
    kw = dict(K=2, level=h.info()["leaf_level"] - 1, kind=hmps.PS_NESTED)
    h.solve(B, **kw)
    torch.cuda.synchronize()
    out = torch.empty_like(d)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.solve(d, out=out, **kw)
    first = x = None
    for rep in range(3):
        print(f"[gpu-case] nested without lists, replay {rep}", flush=True)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        first = got if first is None else first
        assert np.array_equal(got, first), rep
        x = h.solve(d, **kw).cpu().numpy()  # eager: makes the lists
        assert np.linalg.norm(got - x) <= 1e-10 * np.linalg.norm(x), rep
    del g
    h.close()
