"""Batches that wait for room at the same time, none of them running: each is
solved, in pieces where its geometry holds some workspace, else one after the
other (the younger gives its geometry up and is built again)."""
import math
import time

import numpy as np
import pytest

import workloads as W
from parity import assert_close

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu

MB = 1 << 20
PROBS = {k: W.sphere_problem(n, math.sqrt(n / 1536), instance=k) for k, n in ((1, 6000), (2, 5900), (3, 200))}


def _b(key, nrhs, instance):
    return W.plane_waves(PROBS[key].xyz, W.directions(nrhs, 3, instance=instance))


def _resident(srv, nrhs):  # every geometry with the workspace of nrhs right-hand sides
    for key in (1, 2, 3):
        srv.wait(srv.submit(key, _b(key, nrhs, key), K=2, prob=PROBS[key], leaf_max=64))


@pytest.mark.parametrize("gmres", [False, True])
def test_two_batches_wait_for_room(gmres):
    nrhs, held = (16, 16) if gmres else (64, 1)  # no GMRES basis is held at first
    srv = hmps.Server(slots=1)
    _resident(srv, held)
    budget = srv.info()["resident_bytes"] + 24 * MB
    srv.close()
    srv = hmps.Server(budget_bytes=budget, slots=3)
    _resident(srv, held)
    print(f"[gpu-case]   budget {budget / MB:.1f} MB, {srv.info()}", flush=True)
    assert srv.info()["evictions"] == 0
    # all three work for a while, geometry 3 the longest; the wide batches of the
    # other two follow, and find no room while geometry 3 and each other are busy
    kw = dict(K=4, kind=hmps.PS_GMRES, max_passes=200, refine_tol=1e-8) if gmres else dict(K=3)
    busy = [srv.submit(key, _b(key, 1, 9), K=4, kind=hmps.PS_REFINE_FIXED, max_passes=passes, refine_tol=1e-9)
            for key, passes in ((3, 40000), (1, 1000), (2, 1000))]
    while srv.info()["queued"]:
        time.sleep(0.001)
    print(f"[gpu-case] two batches wait for room, gmres={gmres}", flush=True)
    bs = {key: _b(key, nrhs, 20 + key) for key in (1, 2)}
    ts = {key: srv.submit(key, bs[key], **kw) for key in (1, 2)}
    for t in busy[1:]:
        srv.wait(t, timeout_s=60)
    assert srv.poll(busy[0], want_x=False)[2] is None  # still at work
    got = {key: srv.wait(ts[key], timeout_s=60) for key in (1, 2)}
    srv.wait(busy[0], timeout_s=60)
    info = srv.info()
    print(f"[gpu-case]   {info}", flush=True)
    assert info["requests_failed"] == 0 and info["resident_bytes"] <= budget
    srv.close()
    for key in (1, 2):
        h = hmps.HMatrix(PROBS[key], 64, 1.0, 1e-4)
        x, st = h.solve(torch.from_numpy(np.ascontiguousarray(bs[key])).to("cuda"), stats=True, **kw)
        assert_close(got[key][0], x.cpu().numpy(), 1e-6 if gmres else 1e-12)
        assert all(s["diverged"] == 0 for s in got[key][1])
        h.close()
    if gmres:
        assert info["builds"] >= 4  # one was given up and built again
    else:
        assert info["split_batches"] >= 1


def test_gmres_bases_give_way_before_geometries():
    """Room for a wider workspace comes from the GMRES basis that another, idle
    geometry keeps; the geometry stays, and its next GMRES batch is right."""
    gm = dict(K=4, kind=hmps.PS_GMRES, max_passes=200, refine_tol=1e-8)

    def warm(srv):
        for key in (1, 2):
            srv.wait(srv.submit(key, _b(key, 16, key), K=2, prob=PROBS[key], leaf_max=64))
        return srv.wait(srv.submit(1, _b(1, 16, 5), **gm))[0]

    srv = hmps.Server(slots=1)
    warm(srv)
    budget = srv.info()["resident_bytes"] + 24 * MB
    srv.close()
    srv = hmps.Server(budget_bytes=budget, slots=1)
    want = warm(srv)
    before = srv.info()
    print(f"[gpu-case] GMRES bases give way, {before}", flush=True)
    srv.wait(srv.submit(2, _b(2, 24, 6), K=3))
    after = srv.info()
    assert before["evictions"] == after["evictions"] == 0 and after["split_batches"] == 0
    assert after["resident_bytes"] <= budget
    x, st = srv.wait(srv.submit(1, _b(1, 16, 5), **gm))
    assert_close(x, want, 1e-6)
    assert all(s["diverged"] == 0 for s in st)
    srv.close()
