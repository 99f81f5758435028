"""Half-storage lists over the ranges of their piece sizes (96 to 256 half-panel
columns; far pairs in twos, fours and eights): the K terms in one launch against
one launch per term (the same sums, so the same bits), and against the
premultiplied panels, which share no list with them."""
import math
import sys

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


# 512 pairs and fewer, up to 3,583, and beyond; half-panel pieces at both bounds
# and between; the range where pairs come in eights beside wide pieces
@pytest.mark.parametrize("make, leaf, tol", [
    (lambda: W.sphere_problem(1536, 1.0), 64, 1e-4),
    (lambda: W.sphere_problem(6000, math.sqrt(6000 / 1536)), 64, 1e-4),
    (lambda: W.sphere_problem(13241, math.sqrt(13241 / 1536)), 128, 1e-4),
    (lambda: W.sphere_problem(18000, math.sqrt(18000 / 1536)), 128, 1e-4),
    (lambda: W.cube_problem(28, 28 / 16), 128, 1e-5),
], ids=["sphere_1536", "sphere_6000", "sphere_13241", "sphere_18000", "cube_28"])
def test_half_piece_sizes(make, leaf, tol):
    prob = make()
    h = hmps.HMatrix(prob, leaf, 1.0, tol)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    for prec, bar in ((hmps.HM_F64, 1e-12), (hmps.HM_F32_APPLY, 1e-5)):
        got = {}
        for half in (1, 3, 2):
            print(f"[gpu-case] half pieces n={prob.n} precision={prec} half={half}", flush=True)
            sys.stdout.flush()
            h.tune(half_storage=half)
            got[half] = h.solve(d, K=3, precision=prec).cpu().numpy()
        assert np.array_equal(got[1], got[3])
        assert np.linalg.norm(got[1] - got[2]) <= bar * np.linalg.norm(got[2])
    h.close()
