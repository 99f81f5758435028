"""Far factors packed on the device (the default build) against those packed on
the host (HM_BUILD_KEEP_HOST): the operator by the streaming, half-storage and
matrix-core products at every level, on leaves at two depths, a volume, a batch
and blocks whose ranks pass the device's column limits (32, then 128)."""
import math
import sys

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu


def _sphere(n):
    return W.sphere_problem(n, math.sqrt(n / 1536))


def _boxes(k):
    """Four well separated boxes of 180 random points (six far pairs)."""
    p = W.sphere_problem(720, 1.0)
    x = np.random.RandomState(3).uniform(0.0, 1.0, (720, 3))
    x[180:360, 0] += 3.0
    x[360:540, 1] += 3.0
    x[540:, :2] += 3.0
    p.xyz[:] = x
    p.k = k
    return p


@pytest.mark.parametrize("name, make, leaf, tol, bar", [
    # the same rules on both sides: equal to rounding
    ("two_depths", lambda: _sphere(2200), 68, 1e-6, 1e-13),
    ("volume", lambda: W.cube_problem(10, 10 / 16), 32, 1e-5, 1e-13),
    ("batch", lambda: [_sphere(700), W.cube_problem(8, 8 / 16)], 32, 1e-5, 1e-13),
    # oscillatory: ranks of 90 (above the 32 columns of the first pass) and of
    # 180 (above 128: compressed on the host); pivots may differ by rounding,
    # so both sides are within tol of the entries
    ("rank_90", lambda: _boxes(60.0), 200, 1e-6, 1e-4),
    ("rank_180", lambda: _boxes(400.0), 200, 1e-6, 1e-4),
])
def test_far_factors_packed_on_the_device(name, make, leaf, tol, bar):
    prob = make()
    hd = hmps.HMatrix(prob, leaf, 1.0, tol)
    hh = hmps.HMatrix(prob, leaf, 1.0, tol, flags=hmps.HM_BUILD_KEEP_HOST)
    i = hd.info()
    n, top = i["n"], i["leaf_level"]
    ranks = [f["rank_sum"] / f["blocks"] for f in i["far"].values()]
    assert max(ranks) > {"rank_90": 32, "rank_180": 128}.get(name, 0), ranks
    rng = np.random.RandomState(5)
    X = rng.standard_normal((n, 17)) + 1j * rng.standard_normal((n, 17))
    levels = [-1] + [lv for lv in range(max(i["min_far_level"], 0), top)]
    for nrhs in (1, 3, 17):
        x = torch.from_numpy(np.ascontiguousarray(X[:, 0] if nrhs == 1 else X[:, :nrhs])).to("cuda")
        for lev in levels:
            for half in ((1, 2) if nrhs == 1 else (1,)):
                print(f"[gpu-case] pack {name} nrhs={nrhs} level={lev} half={half}", flush=True)
                sys.stdout.flush()
                for h in (hd, hh):
                    h.tune(half_storage=half)
                a, b = (h.apply(x, level=lev).cpu().numpy() for h in (hd, hh))
                assert np.linalg.norm(a - b) <= bar * np.linalg.norm(b), (name, nrhs, lev, half)
    hd.close()
    hh.close()
