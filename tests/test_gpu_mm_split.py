"""The matrix-core term kernel's splits of a workgroup, against the oracle:
leaves on both sides of every row split (64, 96 and 128 rows), right-hand
sides on both sides of every tile width, and work lists from one piece per
leaf to more pieces than one pass of the partial-row sums takes (64)."""
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

TOL_F64 = 1e-10   # the FP64 bar of the other parity tests
TOL_F32 = 1e-4    # the FP32-block bar


# leaf bound, points: leaves of 59/60, 79/80, 96/97, 125/126 and 160/161 rows
@pytest.mark.parametrize("leaf, n", [(64, 953), (80, 1275), (100, 1547), (128, 2010), (170, 2567)])
def test_mm_row_and_column_splits(leaf, n):
    prob = W.sphere_problem(n, math.sqrt(n / 1536))
    H = hmatrix.HMatrix(prob, leaf, 1.0, 1e-4)
    h = hmps.HMatrix(prob, leaf, 1.0, 1e-4)
    B = W.plane_waves(prob.xyz, W.directions(65, 7))
    levels = [-1] + ([min(H.far_levels)] if len(H.far_levels) else [])
    h.tune(mm_min_rhs=1)
    # term_wgs: the default rule, one unit (whole leaves), a unit count that is
    # no multiple of the XCD count, and more units than columns
    for wgs in (-1, 1, 37, 5000):
        h.tune(term_wgs=wgs)
        for nrhs in (1, 5, 16, 17, 33, 48, 65):
            if wgs != -1 and nrhs not in (5, 17, 65):
                continue
            b = torch.from_numpy(np.ascontiguousarray(B[:, :nrhs])).to("cuda")
            for lev in levels:
                print(f"[gpu-case] mm split leaf={leaf} n={n} wgs={wgs} nrhs={nrhs} level={lev}", flush=True)
                sys.stdout.flush()
                ref = series.series(H, B[:, :nrhs], 2, lev)
                for prec, tol in ((hmps.HM_F64, TOL_F64), (hmps.HM_F32_APPLY, TOL_F32)):
                    x = h.solve(b, K=2, level=lev, precision=prec).cpu().numpy()
                    assert_close(x, ref, tol, (wgs, nrhs, lev, prec))
                    again = h.solve(b, K=2, level=lev, precision=prec).cpu().numpy()
                    assert np.array_equal(x, again), (wgs, nrhs, lev, prec)
                y = h.apply(b, level=lev).cpu().numpy()
                assert_close(y, series.apply_Z(H, B[:, :nrhs], lev), 1e-12, (wgs, nrhs, lev))
    h.close()


def test_mm_threshold_default_and_chosen():
    """FP64 products of five to seven right-hand sides take the matrix cores
    only while the threshold is the default; both families agree to rounding."""
    prob = W.sphere_problem(700, math.sqrt(700 / 1536))
    h = hmps.HMatrix(prob, 64, 1.0, 1e-4)
    b = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.directions(7, 2)))).to("cuda")
    assert h.tuning()["mm_min_rhs"] == 8
    x = h.solve(b, K=4).cpu().numpy()
    h.tune(mm_min_rhs=8)           # chosen: streaming kernels for seven
    assert h.tuning()["mm_min_rhs"] == 8
    xs = h.solve(b, K=4).cpu().numpy()
    h.tune(mm_min_rhs=-1)
    assert_close(xs, x, 1e-12)
    assert np.array_equal(h.solve(b, K=4).cpu().numpy(), x)
    h.close()
