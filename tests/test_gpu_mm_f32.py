"""The FP32 matrix-core products (three real ones per complex product, summed in
FP32 within a wave's part) of long lists, for every split of a workgroup: lists
this long are the ones that take them (shorter ones sum FP32 blocks in FP64), so
the handles are batches of one sphere.  Each instance against the FP64 blocks,
per term launches and, where it applies, all terms in one.

The bar is that of FP32 blocks: each entry is off by up to 2^-24 of itself, each
product's sums over c columns by about 2^-24 sqrt(c); four terms over at most
2,048 columns stay below 2e-5 of the norm, well inside the FP32 bar of the other
tests (1e-4)."""
import math
import sys

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
from paper_2307_03968_amd import hmps  # noqa: E402

pytestmark = pytest.mark.gpu

BAR = 2e-5


# leaf bound, points, instances, entries of a series term at least: leaves of 64
# rows past 64 M entries (two units a CU) and past 200 M (eight), of 94, 125 and
# 188 rows past 48 M
@pytest.mark.parametrize("leaf, n, count, entries", [
    (64, 8192, 8, 64e6), (64, 8192, 20, 200e6), (96, 12000, 3, 48e6), (128, 16000, 2, 48e6),
    (200, 12000, 2, 48e6),
], ids=["64_rows", "64_rows_long", "94_rows", "125_rows", "188_rows"])
def test_f32_products_of_long_lists(leaf, n, count, entries):
    probs = [W.sphere_problem(n, math.sqrt(n / 1536), instance=i) for i in range(count)]
    h = hmps.HMatrix(probs, leaf, 1.0, 1e-4, flags=hmps.HM_BUILD_NO_HALF)
    info = h.info()
    assert max(info["series_entries"]) >= entries, max(info["series_entries"])
    small = info["max_leaf"] <= 64
    B = torch.cat([torch.from_numpy(np.ascontiguousarray(W.plane_waves(p.xyz, W.directions(33, 7))))
                   for p in probs]).to("cuda")
    for nrhs in (8, 16, 17, 33):
        b = B[:, :nrhs]
        ref = h.solve(b, K=4)
        for multi in ((2, 1) if small and nrhs <= 32 else (2,)):
            print(f"[gpu-case] FP32 products leaf={leaf} count={count} nrhs={nrhs} multi={multi}", flush=True)
            sys.stdout.flush()
            h.tune(mm_multi=multi)
            x = h.solve(b, K=4, precision=hmps.HM_F32_APPLY)
            for i in range(count):
                rows = slice(int(h.offsets[i]), int(h.offsets[i + 1]))
                err = torch.linalg.vector_norm(x[rows] - ref[rows], dim=0) / torch.linalg.vector_norm(ref[rows], dim=0)
                assert float(err.max()) <= BAR, (nrhs, multi, i, float(err.max()))
                assert float(err.min()) > 0.0  # FP32 blocks did run
            assert torch.equal(x, h.solve(b, K=4, precision=hmps.HM_F32_APPLY))
        h.tune(mm_multi=-1)
    h.close()
