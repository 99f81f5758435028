"""Global far blocks of one right-hand side (t = W_g y_s), against the oracle:
source clusters on both sides of the 1,024 inputs that a workgroup stages at a
time, and row counts that end inside a 32-row (FP64) or 64-row (FP32) tile."""
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


# clusters of the coarsest far level: 256, 1,024 and 1,025 to 1,100 points
@pytest.mark.parametrize("n", [1024, 4096, 4399])
def test_stage_a_one_rhs(n):
    prob = W.sphere_problem(n, math.sqrt(n / 1536))
    H = hmatrix.HMatrix(prob, 64, 1.0, 1e-4)
    h = hmps.HMatrix(prob, 64, 1.0, 1e-4)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    for lev in sorted(set(H.far_levels)):
        ref = series.apply_Z(H, b, lev)
        # FP64 bar of the other products; FP32 blocks round entries to 2^-24
        for prec, tol in ((hmps.HM_F64, 1e-12), (hmps.HM_F32_APPLY, 1e-6)):
            print(f"[gpu-case] stage A n={n} level={lev} precision={prec}", flush=True)
            sys.stdout.flush()
            y = h.apply(d, level=lev, precision=prec).cpu().numpy()
            assert_close(y, ref, tol, (n, lev, prec))
            assert np.array_equal(y, h.apply(d, level=lev, precision=prec).cpu().numpy())
    h.close()
