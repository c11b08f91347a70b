"""The gridder's work queue at the totals where its pops change: up to four
items per workgroup one by one, beyond that four at a time with a remainder
of one to three, for plans and for a batch (one queue over its plans).  512
workgroups run (two per CU on 256 CUs), so single pops end at 2048 items.

Every tile with a visibility is one item here, so the number of items is
exact.  Against the oracle; tolerances as in the other parity tests: FP64
rel-max 1e-12, FP32 rel-L2 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import wstack as o  # noqa: E402
import paper_2301_06061_amd as ws  # noqa: E402
from paper_2301_06061_amd.batch import BatchedImager  # noqa: E402

from test_gpu_parity import assert_close, dev, host  # noqa: E402

pytestmark = pytest.mark.gpu

N, NW, T = 512, 48, 64          # 64 tiles a plane, 3072 in all


def _case(items, precision, seed=0):
    """One to three visibilities inside each of `items` tiles."""
    wl = synth.edge_case(1, n=N, nw=NW, m=64, precision=precision, bad=False)
    p = o.Params.of(wl)
    rng = np.random.default_rng(100 + seed)
    tile = rng.permutation(NW * 64)[:items]
    tile = np.concatenate([tile, rng.choice(tile, items)])
    k, ty, tx = tile // 64, tile // 8 % 8, tile % 8
    m = tile.size
    x = tx * T + rng.uniform(8, T - 8, m)
    y = ty * T + rng.uniform(8, T - 8, m)
    w = o.plane_centres(p)[k]
    assert np.array_equal(o.plane_index(p, w), k)
    wl.uvw = np.stack([(x - N / 2) / wl.fov_l, (y - N / 2) / wl.fov_m, w],
                      axis=1)
    c = rng.standard_normal((2, m))
    wl.vis = (c[0] + 1j * c[1]).astype(wl.vis.dtype)
    wl.weight = rng.uniform(0.5, 1.5, m).astype(np.float32)
    return wl


def _ref(wl):
    return o.image(o.Params.of(wl), wl.uvw, wl.vis, wl.weight)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("items", [1, 511, 2048, 2051, 2052, 2055, 2057,
                                   3072])
def test_queue_totals(items, precision):
    wl = _case(items, precision)
    ref = _ref(wl)
    plan = ws.WStackPlan.from_workload(wl)
    for _ in range(2):
        assert_close(host(plan.dirty_image(*dev(wl))), ref, precision == 1,
                     f"{items} items")
    plan.close()


@pytest.mark.parametrize("items", [(3, 2048), (1030, 1025), (3072, 1)])
def test_queue_of_a_batch(items):
    wls = [_case(n, 0, seed) for seed, n in enumerate(items)]
    b = BatchedImager(wls, *zip(*(dev(wl) for wl in wls)), precision="fp32")
    for img, wl in zip(b.run(), wls):
        assert_close(host(img), _ref(wl), False, f"batch of {items}")
    b.close()
