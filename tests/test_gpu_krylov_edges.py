"""The vector kernels of GMRES at their edges, against the oracle's x*: rows on
both sides of a 256-row workgroup, one vector and more than a wave's share of
vectors, the longest cycle (64 steps, run to the end by a tolerance that is
not reached), one and several right-hand sides, one of them zero."""
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

TOL_X = 1e-8      # the bar of the other GMRES tests, for
RES_TOL = 1e-11   # this residual tolerance


@pytest.mark.parametrize("n", [40, 255, 256, 257, 1025])
def test_gmres_vector_kernels(n):
    prob = W.sphere_problem(n, math.sqrt(n / 1536))
    H = hmatrix.HMatrix(prob, 32, 1.0, 1e-6)
    h = hmps.HMatrix(prob, 32, 1.0, 1e-6)
    B = W.plane_waves(prob.xyz, W.directions(3, 5))
    B[:, 1] = 0.0
    xs = series.solve_exact(H, B[:, [0, 2]], -1)
    for nrhs, cols in ((1, [0]), (3, [0, 1, 2])):
        b = torch.from_numpy(np.ascontiguousarray(B[:, 0] if nrhs == 1 else B)).to("cuda")
        for K, restart, passes, tol in ((0, 7, 300, RES_TOL), (0, 64, 300, RES_TOL),
                                        (2, 0, 300, RES_TOL), (0, 64, 64, 1e-30)):
            print(f"[gpu-case] gmres n={n} nrhs={nrhs} K={K} restart={restart} tol={tol}", flush=True)
            sys.stdout.flush()
            kw = dict(K=K, kind=hmps.PS_GMRES, restart=restart, max_passes=passes, refine_tol=tol)
            x, st = h.solve(b, stats=True, **kw)
            x = x.cpu().numpy().reshape(n, nrhs)
            assert_close(x[:, 0], xs[:, 0], TOL_X, (n, nrhs, K, restart))
            if nrhs == 3:
                assert_close(x[:, 2], xs[:, 1], TOL_X, (n, nrhs, K, restart))
                assert not x[:, 1].any()
            if tol == RES_TOL:
                assert all(s["resid_rel"] <= RES_TOL for s in st), st
            again = h.solve(b, **kw).cpu().numpy().reshape(n, nrhs)
            assert np.array_equal(x, again)
    h.close()
