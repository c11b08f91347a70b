"""The fused row kernels over the shapes where their launch changes: planes
of one row transformed by 1, 2, 4 or 8 groups of a workgroup (images of few
rows), plane counts that do not divide into the groups, degridding's planes
cut into runs, rows of 64 to 8192 points, and sparse images whose tiles
without records stay unwritten (the stack starts as NaN) on small grids too.

Against the oracle; tolerances as in the other parity tests: FP64 rel-max
1e-12, FP32 rel-L2 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import wstack as o  # noqa: E402
import paper_2301_06061_amd as ws  # noqa: E402

from test_gpu_parity import assert_close, dev, host  # noqa: E402

pytestmark = pytest.mark.gpu

SHAPES = [
    (64, 64, 1), (64, 64, 2), (64, 128, 3), (128, 64, 9), (256, 256, 5),
    (256, 4096, 3), (512, 128, 9), (512, 512, 17), (1024, 128, 7),
    (1024, 2048, 2), (2048, 64, 3), (2048, 1024, 2), (4096, 64, 5),
    (8192, 64, 3), (64, 8192, 2),
]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nu,nv,nw", SHAPES)
def test_row_shapes(nu, nv, nw, precision):
    fp64 = precision == "fp64"
    wl = synth.random_case(90 + nw, n=nu, nv=nv, nw=nw, support=7, m=150,
                           law="gauss", fov_deg=0.1,
                           precision=1 if fp64 else 0)
    p = o.Params.of(wl)
    ref = o.image(p, wl.uvw, wl.vis, wl.weight)
    uvw, vis, wt = dev(wl)
    plan = ws.WStackPlan.from_workload(wl)
    plan.planes.fill_(complex(float("nan"), float("nan")))
    img = plan.dirty_image(uvw, vis, wt)
    assert_close(host(img), ref, fp64, "one call")
    plan.reset()
    plan.grid(uvw, vis, wt)
    img2 = plan.new_image()
    plan.image_accumulate(img2)
    assert_close(host(img2), ref, fp64, "two calls")
    x = np.random.default_rng(2).standard_normal((nv, nu))
    v = plan.degrid(torch.from_numpy(x).to("cuda").to(plan.rdtype), uvw, wt)
    assert_close(host(v), o.degrid(p, x, wl.uvw, wl.weight), fp64, "degrid")
    plan.close()
