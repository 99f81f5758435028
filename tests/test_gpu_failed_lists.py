"""A rebuild of the work lists that fails (the upload refused by a hook): calls
that would run on the lists are refused until a rebuild succeeds, and results
are then as before."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [1, 4, 20])
def test_failed_rebuild_is_refused_until_mended(nrhs):
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.directions(nrhs, 3)))).to("cuda")
    x = h.solve(b, K=2).cpu().numpy()
    assert hmps._lib().hm_debug_fail_lists(h.handle) == hmps.HM_OK
    with pytest.raises(Exception, match="work lists failed"):
        h.tune(term_wgs=37)
    print(f"[gpu-case] calls after a failed rebuild, nrhs={nrhs} (refused)", flush=True)
    for call in (lambda: h.solve(b, K=2), lambda: h.apply(b),
                 lambda: h.solve(b, K=1, kind=hmps.PS_NESTED)):
        with pytest.raises(Exception, match="work lists are missing"):
            call()
    h.tune(term_wgs=37)  # the same value again: built now
    y = h.solve(b, K=2).cpu().numpy()
    assert np.linalg.norm(y - x) <= 1e-12 * np.linalg.norm(x)
    h.tune(term_wgs=-1)
    assert np.array_equal(h.solve(b, K=2).cpu().numpy(), x)
    h.close()


def test_failed_level_list_is_made_by_the_next_call():
    prob = W.sphere_problem(1200, math.sqrt(1200 / 1536))
    h = hmps.HMatrix(prob, 32, 1.0, 1e-4)
    b = W.plane_waves(prob.xyz, W.directions(1, 3)).reshape(-1)
    d = torch.from_numpy(np.ascontiguousarray(b)).to("cuda")
    kw = dict(K=2, level=h.info()["leaf_level"] - 1, kind=hmps.PS_NESTED)
    h.solve(d, K=2)
    assert hmps._lib().hm_debug_fail_lists(h.handle) == hmps.HM_OK
    with pytest.raises(Exception, match="work lists failed"):
        h.solve(d, **kw)
    print("[gpu-case] nested solve after a failed level list", flush=True)
    x = h.solve(d, **kw).cpu().numpy()
    h.tune(half_storage=2)
    ref = h.solve(d, **kw).cpu().numpy()
    assert np.linalg.norm(x - ref) <= 1e-10 * np.linalg.norm(ref)
    h.close()
