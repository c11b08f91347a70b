"""Batches of several plans whose idle tiles are zeroed (tile edges 16 and 32,
different tile counts) before, between and after plans that leave theirs
unwritten (tile edge 64).

Every stack is filled with NaN first, so that an idle tile the batched
zeroing misses, or takes from another plan's list, reaches the image.
Images against the oracle on two runs (the second meets the first's stacks)
and on graph replays; FP64 rel-max 1e-12, FP32 rel-L2 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import wstack as o  # noqa: E402
from paper_2301_06061_amd.batch import BatchedImager  # noqa: E402

from test_gpu_parity import assert_close, host  # noqa: E402

pytestmark = pytest.mark.gpu

# (n, nv, nw, m, tile)
PLANS = [(128, 128, 3, 60, 16),      # 192 tiles
         (256, 256, 2, 400, 64),
         (256, 128, 5, 90, 32),      # 160 tiles
         (64, 64, 1, 0, 16),         # 16 tiles, all idle
         (128, 256, 2, 70, 16),      # 256 tiles
         (512, 512, 2, 300, 64),
         (512, 256, 3, 500, 32)]     # 384 tiles


def _workloads(precision, order):
    out = []
    for i in order:
        n, nv, nw, m, _ = PLANS[i]
        wl = synth.random_case(60 + i, n=n, nv=nv, nw=nw, support=7,
                               m=max(m, 1), law="core",
                               precision=1 if precision == "fp64" else 0)
        if m == 0:
            wl.uvw, wl.vis, wl.weight = wl.uvw[:0], wl.vis[:0], wl.weight[:0]
        if nw == 1:
            wl.w_max = wl.w_min
        out.append(wl)
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("order", [(0, 1, 2, 3, 4, 5, 6),
                                   (5, 6, 4, 0, 3, 2, 1),
                                   (3, 0), (2, 6, 0)])
def test_zeroed_plans_in_a_batch(order, precision):
    fp64 = precision == "fp64"
    wls = _workloads(precision, order)
    dev = [[torch.from_numpy(np.ascontiguousarray(getattr(w, k))).cuda()
            for w in wls] for k in ("uvw", "vis", "weight")]
    refs = [o.image(o.Params.of(w), w.uvw, w.vis, w.weight) for w in wls]
    b = BatchedImager(wls, *dev, precision=precision,
                      params=[(PLANS[i][4], 0) for i in order])

    def poison():
        for p in b.plans:
            p.planes.fill_(float("nan"))
        torch.cuda.synchronize()

    def check(images, scale, what):
        for i, img, ref in zip(order, images, refs):
            got = host(img)
            if not np.any(ref):
                assert not np.any(got), (what, i)
            else:
                assert_close(got, ref * scale, fp64, f"{what} plan {i}")

    poison()
    check(b.run(), 1.0, "first run")
    check(b.run(), 1.0, "second run")
    b.capture()
    for rep in range(3):
        if rep != 1:
            poison()
        for v, w in zip(dev[1], wls):
            v.copy_(torch.from_numpy(w.vis).cuda() * (rep + 1.0))
        torch.cuda.synchronize()
        check(b.replay(), rep + 1.0, f"replay {rep}")
    b.close()
