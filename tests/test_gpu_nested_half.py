"""The nested solve of one right-hand side in the scaled basis, against the
oracle's ``nested``: leaves at one depth and at two (in-row far blocks whose
first row of a level is odd), a surface and a volume, every level, with the
leaf-level factor in one launch and in one per term, and after the work lists
are rebuilt.  Bars as for the other nested parity tests."""
import math
import sys

import numpy as np
import pytest

import workloads as W
from oracle import hmatrix, series
from parity import assert_close

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu

TOL_F64 = 1e-10
TOL_F32 = 1e-4


def _sphere(n):
    return W.sphere_problem(n, math.sqrt(n / 1536))


@pytest.mark.parametrize("name, make, leaf, tol", [
    ("sphere_1200", lambda: _sphere(1200), 32, 1e-6),
    ("sphere_2200_two_depths", lambda: _sphere(2200), 68, 1e-4),
    ("cube_1000", lambda: W.cube_problem(10, 10 / 16), 32, 1e-5),
])
def test_nested_one_rhs(name, make, leaf, tol):
    prob = make()
    H = hmatrix.HMatrix(prob, leaf, 1.0, tol)
    h = hmps.HMatrix(prob, leaf, 1.0, tol)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")

    def solve(lev, K, prec):
        print(f"[gpu-case] nested one RHS {name} level={lev} K={K} precision={prec}", flush=True)
        sys.stdout.flush()
        return h.solve(d, K=K, level=lev, precision=prec, kind=hmps.PS_NESTED).cpu().numpy()

    for lev in [-1] + sorted(H.far_levels, reverse=True):
        for K in (0, 1, 2, 3):
            if K == 3 and len([q for q in H.far_levels if q >= lev]) > 3:
                continue  # (K + 1)^levels products
            ref = series.nested(H, b, K, lev)
            for prec, bar in ((hmps.HM_F64, TOL_F64), (hmps.HM_F32_APPLY, TOL_F32)):
                x = solve(lev, K, prec)
                assert_close(x, ref, bar, (name, lev, K, prec))
                assert np.array_equal(x, solve(lev, K, prec))
    # per-term launches, panels (no half storage) and rebuilt lists
    lo = sorted(H.far_levels)[-2] if len(H.far_levels) > 1 else min(H.far_levels)
    ref = series.nested(H, b, 2, lo)
    for tuning in (dict(half_storage=3), dict(half_storage=2), dict(half_storage=-1),
                   dict(term_wgs=37), dict(term_wgs=-1)):
        h.tune(**tuning)
        assert_close(solve(lo, 2, hmps.HM_F64), ref, TOL_F64, tuning)
    h.close()


def test_nested_one_rhs_captured():
    """A captured nested solve replays to the eager result."""
    prob = _sphere(1200)
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    kw = dict(K=2, level=h.info()["leaf_level"] - 1, kind=hmps.PS_NESTED)
    x = h.solve(d, **kw).cpu().numpy()
    out = torch.empty_like(d)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        h.solve(d, out=out, **kw)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.solve(d, out=out, **kw)
    for rep in range(3):
        print(f"[gpu-case] nested one RHS, replay {rep}", flush=True)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), x), rep
        h.solve(d, **kw).cpu()  # eager work between replays
    del g
    h.close()
