"""Degridding of tiles just below, at and above the sizes where its kernel
changes: up to 32 records read from the plane directly, more from the staged
tile (one to four records a thread and beyond, several items), with the
nearest cells on tile borders, grid edges and off the grid, for every kernel
support and both stack row orders (columns beyond 4096 leave rows in
four-step order).

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


def _tile_case(n, nv, support, counts, precision):
    """counts[t] visibilities in tile t (row-major), two thirds of them
    within the halo of a tile border, plus a few off every grid edge."""
    # (A tall grid gets a narrow field: fov_m = fov_l nv / n.)
    wl = synth.edge_case(3, n=n, nv=nv, nw=1, support=support, m=64,
                         fov_deg=2.0 if nv <= 4 * n else 0.1,
                         precision=precision, bad=False)
    rng = np.random.default_rng(11)
    T = min(64, n, nv)
    h = (support - 1) // 2
    xs, ys = [], []
    for t, c in enumerate(counts):
        ty, tx = divmod(t, n // T)
        u = rng.integers(0, T, (c, 2)).astype(float)
        edge = rng.random((c, 2)) < 0.4
        near = rng.integers(0, h + 1, (c, 2)) + (T - 1 - h) * rng.integers(
            0, 2, (c, 2))
        u = np.where(edge, np.clip(near, 0, T - 1), u)
        f = rng.uniform(-0.49, 0.49, (c, 2))
        xs.append(tx * T + u[:, 0] + f[:, 0])
        ys.append(ty * T + u[:, 1] + f[:, 1])
    x, y = np.concatenate(xs), np.concatenate(ys)
    uvw = np.stack([(x - n / 2) / wl.fov_l, (y - nv / 2) / wl.fov_m,
                    np.zeros(x.size)], axis=1)
    wl.uvw = np.ascontiguousarray(np.concatenate([wl.uvw, uvw]))
    m = wl.uvw.shape[0]
    wl.vis = np.resize(wl.vis, m)
    wl.weight = rng.uniform(0.5, 1.5, m).astype(np.float32)
    return wl


COUNTS = [1, 31, 32, 33, 0, 9, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025,
          1300]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("support", [1, 3, 5, 7, 9, 11, 13, 15])
def test_degrid_tile_sizes(support, precision):
    wl = _tile_case(256, 256, support, COUNTS, 1 if precision == "fp64" else 0)
    _check(wl, precision == "fp64")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nv,support", [(32, 32, 7), (16, 64, 5),
                                          (64, 8192, 9)])
def test_degrid_other_tiles(n, nv, support, precision):
    T = min(64, n, nv)
    tiles = (n // T) * (nv // T)
    wl = _tile_case(n, nv, support, COUNTS[:tiles],
                    1 if precision == "fp64" else 0)
    _check(wl, precision == "fp64")


def _check(wl, fp64):
    p = o.Params.of(wl)
    x = np.random.default_rng(5).standard_normal((wl.nv, wl.nu))
    ref = o.degrid(p, x, wl.uvw, wl.weight)
    uvw, _, wt = dev(wl)
    for chunk in (0, 40):
        plan = ws.WStackPlan.from_workload(wl, chunk=chunk)
        v = plan.degrid(torch.from_numpy(x).to("cuda").to(plan.rdtype), uvw,
                        wt)
        assert_close(host(v), ref, fp64, f"chunk {chunk}")
        plan.close()
