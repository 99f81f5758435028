"""A tuning read and written back, at once or after other values, is the same
tuning: the same kernels and so the same bits, on both sides of the FP64 and
FP32 thresholds of the matrix cores."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 4, 5, 7, 8])
def test_tuning_read_and_written_back(nrhs):
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.directions(nrhs, 3)))).to("cuda")

    def solves():
        print(f"[gpu-case] tuning round trip, nrhs={nrhs}", flush=True)
        return [h.solve(b, K=3, precision=p).cpu().numpy() for p in (hmps.HM_F64, hmps.HM_F32_APPLY)]

    want, t = solves(), h.tuning()
    h.tune(**t)
    assert h.tuning() == t
    assert all(np.array_equal(x, y) for x, y in zip(solves(), want))
    # streaming kernels, then matrix cores for every width, then back
    for other in (64, 1):
        h.tune(mm_min_rhs=other)
        for x, y in zip(solves(), want):
            assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y)
        h.tune(**t)
        assert all(np.array_equal(x, y) for x, y in zip(solves(), want))
    h.close()


def test_autotuned_tuning_written_back():
    """What the autotuner chose for seven right-hand sides says which kernels
    run: the same bits with the default restored and the choice written back."""
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.directions(7, 3)))).to("cuda")
    best, _ = h.autotune(7, K=3)
    assert best["mm_min_rhs"] == 7 or best["mm_min_rhs"] == 9
    want, t = h.solve(b, K=3).cpu().numpy(), h.tuning()
    h.tune(mm_min_rhs=-1, term_wgs=-1, rhs_tile=-1, inrow_pct=-1, half_storage=-1, mm_multi=-1)
    h.solve(b, K=3)
    h.tune(**t)
    assert np.array_equal(h.solve(b, K=3).cpu().numpy(), want)
    h.close()
