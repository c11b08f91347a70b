"""The direct sort and single-workgroup scans of small plans
(binning="auto") against the two-level partition and the oracle, at the
edges of their blocks: one visibility, whole counting workgroups and one
more, the sizes where the counting block, the scan and the sort itself
change, rows of several channels, slabs, empty calls, degridding.

Both sorts give the same records per key, so the tile statistics are equal
(exactly); images differ by the order of FP additions only.  Tolerances as
in the other parity tests: FP64 rel-max 1e-12, FP32 rel-L2 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import wstack as o  # noqa: E402
import paper_2301_06061_amd as ws  # noqa: E402

pytestmark = pytest.mark.gpu


def _dev(wl):
    d = torch.device("cuda", 0)
    wt = None if wl.weight is None else torch.from_numpy(wl.weight).to(d)
    return (torch.from_numpy(np.ascontiguousarray(wl.uvw)).to(d),
            torch.from_numpy(np.ascontiguousarray(wl.vis)).to(d), wt)


def _err(a, b, fp64):
    a, b = a.to(torch.complex128), b.to(torch.complex128)
    if not bool((b != 0).any()):
        return float(a.abs().max())
    if fp64:
        return float((a - b).abs().max() / b.abs().max())
    return float(torch.linalg.vector_norm(a - b) /
                 torch.linalg.vector_norm(b))


# (n, nv, nw, m): counting blocks of 1024 and 4096, key totals inside the
# tile work pass or in a kernel of their own (65536 histogram words), 16384
# keys, the level-1 scan in one workgroup (65536 words) and not.
SIZES = [
    (64, 64, 1, 1),
    (64, 64, 3, 1024),
    (128, 128, 4, 1025),
    (32, 16, 2, 4095),
    (256, 256, 8, 57_000),       # 1152 keys x 56 blocks <= 65536
    (256, 256, 8, 58_400),       # 58 blocks: past it
    (128, 256, 5, 65_536),
    (128, 256, 5, 65_537),       # large counting blocks
    (512, 512, 28, 9_000),       # 16128 keys
    (512, 512, 29, 9_000),       # 16704: the partition, one-workgroup scan
    (512, 1024, 40, 300_000),    # 640 buckets x 74 blocks <= 65536
    (512, 1024, 64, 300_000),    # 1024 x 74: past it
]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nv,nw,m", SIZES)
def test_small_plan_sort_equals_partition(n, nv, nw, m, precision):
    fp64 = precision == "fp64"
    tol = 1e-12 if fp64 else 1e-5
    sup = 5 if min(n, nv) < 32 else 7
    wl = synth.edge_case(7, n=n, nv=nv, nw=nw, support=sup, m=m,
                         precision=1 if fp64 else 0)
    uvw, vis, wt = _dev(wl)
    x = np.random.default_rng(1).standard_normal((nv, n))
    out = {}
    for mode in ("auto", "partition"):
        plan = ws.WStackPlan.from_workload(wl, binning=mode)
        drop = torch.zeros(1, dtype=torch.int64, device="cuda")
        img = plan.dirty_image(uvw, vis, wt, dropped=drop)
        stats = plan.tile_stats()
        # Slabs: the second call adds to what the first wrote.
        plan.reset()
        cut = m // 3
        plan.grid(uvw[:cut], vis[:cut], wt[:cut])
        plan.grid(uvw[cut:], vis[cut:], wt[cut:])
        two = plan.new_image()
        plan.image_accumulate(two)
        v = plan.degrid(torch.from_numpy(x).to("cuda").to(plan.rdtype), uvw,
                        wt)
        plan.grid(uvw[:0], vis[:0], wt[:0])  # nothing: an all-zero stack
        none = plan.new_image()
        plan.image_accumulate(none)
        torch.cuda.synchronize()
        assert not bool((none != 0).any())
        out[mode] = (img, two, v, stats, int(drop.item()))
        plan.close()
    a, b = out["auto"], out["partition"]
    assert a[3] == b[3] and a[4] == b[4]
    for i in range(3):
        assert _err(a[i], b[i], fp64) <= tol
    assert _err(a[0], a[1], fp64) <= tol
    if n * nv * nw <= 128 * 256 * 5 or m <= 1025:
        p = o.Params.of(wl)
        ref = torch.from_numpy(o.image(p, wl.uvw, wl.vis, wl.weight))
        assert _err(a[0].cpu(), ref, fp64) <= tol
        vref = torch.from_numpy(o.degrid(p, x, wl.uvw, wl.weight))
        assert _err(a[2].cpu(), vref, fp64) <= tol
