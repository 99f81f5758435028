"""Device memory of a build: the compressed far factors are gone once the
panels are packed, so that no phase after that holds more than the finished
handle, and a server build that waits for room holds none."""
import math
import sys
import time

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def _far_bytes(info):  # U and V of one orientation of each far block
    return 16 * sum(f["entries"] for f in info["far"].values()) // 2


@pytest.mark.parametrize("make, leaf, tol, flags", [
    (lambda: W.sphere_problem(24576, 4.0), 128, 1e-4, 0),
    (lambda: W.sphere_problem(24576, 4.0), 128, 1e-4, hmps.HM_BUILD_NO_HALF),
    (lambda: W.cube_problem(24, 24 / 16), 256, 1e-5, 0),  # leaves past the half storage's bound
], ids=["half", "no_half", "large_leaves"])
def test_build_peak_is_the_handle(make, leaf, tol, flags):
    prob = make()
    hmps.HMatrix(W.sphere_problem(600, 0.625), 64, 1.0, 1e-4).close()  # the code objects are loaded
    marks = []
    base = _used()
    print(f"[gpu-case] build memory n={prob.n} flags={flags}", flush=True)
    h = hmps.HMatrix(prob, leaf, 1.0, tol, flags=flags, progress=lambda m: marks.append((m, _used() - base)))
    end = _used() - base
    far = _far_bytes(h.info())
    for m, u in marks:
        print(f"[gpu-case]   {m}: {u / MB:.1f} MB", flush=True)
    print(f"[gpu-case]   end {end / MB:.1f} MB, far factors {far / MB:.1f} MB", flush=True)
    assert far > 32 * MB
    first = [m for m, _ in marks].index("panels packed and uploaded")
    for m, u in marks[first:]:
        assert u <= end + 8 * MB, (m, u, end)
    # what the handle says it holds is what the device has given out (blocks
    # come in 2 MB pages)
    held = h.info()["device_bytes"]
    assert abs(held - end) <= 24 * MB, (held, end)
    h.close()


@pytest.mark.parametrize("flags", [0, hmps.HM_BUILD_NO_HALF], ids=["half", "no_half"])
def test_build_that_just_fits(flags):
    """With memory for the finished handle and half the far factors, the handle
    is built, with the same result."""
    prob = W.sphere_problem(24576, 4.0)
    b = torch.from_numpy(np.ascontiguousarray(W.plane_waves(prob.xyz, W.Z_HAT).reshape(-1))).to("cuda")
    base = _used()
    h = hmps.HMatrix(prob, 128, 1.0, 1e-4, flags=flags)
    end, far = _used() - base, _far_bytes(h.info())
    x = h.solve(b, K=2).cpu().numpy()
    h.close()
    free, _ = torch.cuda.mem_get_info()
    fill = torch.empty(free - end - far // 2, dtype=torch.uint8, device="cuda")
    print(f"[gpu-case] build of {end / MB:.0f} MB in {torch.cuda.mem_get_info()[0] / MB:.0f} MB, flags={flags}", flush=True)
    h = hmps.HMatrix(prob, 128, 1.0, 1e-4, flags=flags)
    del fill
    torch.cuda.empty_cache()
    assert np.array_equal(h.solve(b, K=2).cpu().numpy(), x)
    h.close()


def test_server_resident_bytes_are_what_the_device_gave_out():
    """Workspace and GMRES basis (32 right-hand sides: 96 and 192 MB) included."""
    srv = hmps.Server(slots=1)

    def requests(key, n):
        p = W.sphere_problem(n, math.sqrt(n / 1536))
        B = W.plane_waves(p.xyz, W.directions(32, 3))
        print(f"[gpu-case] server resident bytes, {n} points", flush=True)
        srv.wait(srv.submit(key, B, K=2, prob=p, leaf_max=64))
        srv.wait(srv.submit(key, B, K=0, kind=hmps.PS_GMRES, max_passes=4, refine_tol=1e-9))
        return _used(), srv.info()["resident_bytes"]

    u0, r0 = requests(1, 600)  # what the kernels' queues need is there from now on
    u1, r1 = requests(2, 6000)
    print(f"[gpu-case]   used {(u1 - u0) / MB:.1f} MB, resident {(r1 - r0) / MB:.1f} MB", flush=True)
    assert abs((u1 - u0) - (r1 - r0)) <= 32 * MB
    srv.close()


@pytest.mark.parametrize("make, leaf, tol", [
    (lambda: W.sphere_problem(6000, math.sqrt(6000 / 1536)), 64, 1e-4),
    (lambda: W.sphere_problem(24576, 4.0), 128, 1e-4),
    (lambda: W.cube_problem(17, 17 / 16), 128, 1e-5),
], ids=["leaf_64", "leaf_128", "volume"])
def test_server_builds_what_it_can_serve(make, leaf, tol):
    """Around the budget that a geometry and its first batch need, a server
    either serves the batch or refuses it before the build; a twentieth more is
    enough."""
    prob = make()
    B = W.plane_waves(prob.xyz, W.directions(64, 3))
    staging = 2 * 16 * 64 * prob.n  # of the worker

    def serve(budget):
        srv = hmps.Server(budget_bytes=budget, slots=1)
        err = None
        try:
            srv.wait(srv.submit(1, B, K=1, prob=prob, leaf_max=leaf, aca_tol=tol))
        except hmps.HmpsError as e:
            err = str(e)
        i = srv.info()
        srv.close()
        return err, i

    need = serve(0)[1]["resident_bytes"] - staging
    got = []
    for pct in range(90, 104):
        budget = need * pct // 100
        print(f"[gpu-case] n={prob.n}, {pct}% of the bytes needed", flush=True)
        err, i = serve(budget)
        got.append((pct, err, i["builds"]))
        assert (i["builds"] == 1 and i["resident_bytes"] <= budget + staging) if err is None else i["builds"] == 0, got[-1]
    assert got[0][1] is not None
    assert serve(need * 105 // 100)[0] is None


def test_server_build_waiting_for_room_holds_no_device_memory():
    """One worker: geometry 2's build has no room while geometry 1 has queued
    requests, so it steps aside; while they run, the device holds geometry 1."""
    p1 = W.sphere_problem(6000, math.sqrt(6000 / 1536))
    p2 = W.sphere_problem(24576, 4.0)
    probe = hmps.HMatrix(p2, 128, 1.0, 1e-4)
    info = probe.info()
    far, big = _far_bytes(info), info["device_bytes"]
    b2 = W.plane_waves(p2.xyz, W.Z_HAT)
    d2 = torch.from_numpy(np.ascontiguousarray(b2.reshape(-1))).to("cuda")
    ref = probe.solve(d2, K=2).cpu().numpy()
    probe.close()
    # geometry 1 with its workspace, as the server counts it
    b1 = W.plane_waves(p1.xyz, W.Z_HAT)
    kw = dict(K=4, kind=hmps.PS_REFINE_FIXED, refine_tol=1e-9)
    srv = hmps.Server(slots=1)
    srv.wait(srv.submit(1, b1, prob=p1, leaf_max=64, max_passes=2, **kw))
    small = srv.info()["resident_bytes"]
    srv.close()
    # geometry 2 fits alone, not beside geometry 1
    srv = hmps.Server(budget_bytes=int(big + 0.7 * small), slots=1)
    srv.wait(srv.submit(1, b1, prob=p1, leaf_max=64, max_passes=2, **kw))
    base = _used_now()
    t2 = srv.submit(2, b2, K=2, prob=p2, leaf_max=128)
    t1 = srv.submit(1, b1, max_passes=8000, **kw)  # about a second and a half
    print(f"[gpu-case] build aside: far factors {far / MB:.1f} MB", flush=True)
    sys.stdout.flush()
    seen = []
    while srv.info()["queued"] > 1 or srv.info()["builds"] < 1:
        time.sleep(0.01)
    while srv.poll(t1, want_x=False)[2] is None:
        i = srv.info()
        if i["queued"] == 1 and i["batches"] == 2 and i["builds"] == 1:
            seen.append(_used_now() - base)
        time.sleep(0.02)
    x2, _ = srv.wait(t2)
    srv.close()
    print(f"[gpu-case]   beside geometry 1: {[round(u / MB, 1) for u in seen[:40]]}", flush=True)
    assert len(seen) >= 4
    assert min(seen) <= far // 2, (min(seen), far)
    assert np.array_equal(np.asarray(x2).reshape(-1), ref)


def _used_now():  # without waiting for the device: a solve runs meanwhile
    free, total = torch.cuda.mem_get_info()
    return total - free
