"""A multi-term launch whose dependency wait gave up is reported, once, by the
next call of every kind that synchronises.  The flagged call has K = 0, so
that no wait runs with the flag set."""
import ctypes as C
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(kind=hmps.PS_SERIES), dict(kind=hmps.PS_NESTED),
    dict(kind=hmps.PS_REFINE_FIXED, max_passes=2, refine_tol=1.0),
    dict(kind=hmps.PS_GMRES, max_passes=40, refine_tol=1e-8),
], ids=["series", "nested", "refine", "gmres"])
def test_give_up_is_reported(kw):
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    kw = dict(kw, level=h.info()["leaf_level"] - 1 if kw["kind"] == hmps.PS_NESTED else -1)
    x = h.solve(d, K=2, stats=True, **kw)[0].cpu().numpy()
    assert hmps._lib().hm_debug_gave_up(h.handle) == hmps.HM_OK
    print(f"[gpu-case] give-up flag set before {kw}", flush=True)
    for _ in range(2):  # the half-storage flag, then the matrix-core launch's
        with pytest.raises(Exception, match="gave up"):
            h.solve(d, K=0, stats=True, **kw)
    assert np.array_equal(h.solve(d, K=2, stats=True, **kw)[0].cpu().numpy(), x)
    h.close()


def test_gave_up_hook_takes_device_handles_only():
    assert hmps._lib().hm_debug_gave_up(C.c_void_p()) == hmps.HM_EINVAL
