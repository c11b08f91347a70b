"""Automatic work items against items of 4096 records: no image takes longer
with them, for narrow and wide kernels, dense cores (on a corner of four
tiles, each read up to four times) and uniform coverage, and the images agree.
"""
import math

import pytest

torch = pytest.importorskip("torch")

import paper_2301_06061_amd as ws  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [(128, 5, 155_209, "core", 1, "fp64"),
         (256, 6, 132_328, "uniform", 1, "fp32"),
         (128, 5, 155_209, "core", 3, "fp64"),
         (512, 8, 200_000, "core", 5, "fp64"),
         (128, 5, 155_209, "core", 15, "fp64"),
         (128, 4, 60_000, "point", 7, "fp32"),
         (256, 8, 30_000, "point", 9, "fp32"),
         (512, 8, 200_000, "core", 15, "fp32"),
         (512, 8, 200_000, "core", 9, "fp64"),
         (1024, 16, 1_000_000, "core", 7, "fp32")]


def _inputs(n, m, law, precision):
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    f64 = dict(generator=g, device="cuda", dtype=torch.float64)
    if law == "uniform":
        xy = (torch.rand(m, 2, **f64) - 0.5) * (n - 16)
    else:
        r = (n / 2 - 8) * torch.rand(m, **f64) ** 2 if law == "core" else \
            2.0 * torch.rand(m, **f64)
        th = torch.rand(m, **f64) * 2 * math.pi
        xy = torch.stack([r * torch.cos(th), r * torch.sin(th)], 1)
    w = torch.rand(m, 1, **f64) * 100 - 50
    vis = torch.randn(m, generator=g, device="cuda",
                      dtype=torch.complex128 if precision == "fp64"
                      else torch.complex64)
    return torch.cat([xy / 0.03, w], 1).contiguous(), vis


def _timed(n, nw, m, K, precision, chunk, uvw, vis):
    plan = ws.WStackPlan(n, n, nw, 0.03, 0.03, -50.0, 50.0, K,
                         precision=precision, max_vis=m, chunk=chunk)
    img, best = plan.dirty_image(uvw, vis), math.inf
    for _ in range(10):
        a = torch.cuda.Event(enable_timing=True)
        b = torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(3):
            plan.dirty_image(uvw, vis)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 3)
    plan.close()
    return img, best


@pytest.mark.parametrize("n,nw,m,law,K,precision", CASES)
def test_no_slower_than_items_of_4096(n, nw, m, law, K, precision):
    uvw, vis = _inputs(n, m, law, precision)
    got, t = _timed(n, nw, m, K, precision, 0, uvw, vis)
    ref, t_ref = _timed(n, nw, m, K, precision, 4096, uvw, vis)
    err = float(torch.linalg.vector_norm(got - ref) /
                torch.linalg.vector_norm(ref))
    assert err <= (1e-13 if precision == "fp64" else 1e-6), err
    assert t <= 1.2 * t_ref, (t, t_ref)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("m,chunk", [(3_000, 16), (9_000, 16), (20_000, 7)])
def test_slots_run_out(m, chunk, precision):
    """All visibilities about the origin, each read by four tiles, in items
    that would need four slots a chunk where two are reserved: the direct sort
    takes larger items.  Image, slabs and statistics against the hashed sort
    with items of 4096."""
    n, nw, K = 128, 2, 7
    uvw, vis = _inputs(n, m, "point", precision)
    out = []
    for binning, c in (("auto", chunk), ("hashed", 4096)):
        plan = ws.WStackPlan(n, n, nw, 0.03, 0.03, -50.0, 50.0, K,
                             precision=precision, max_vis=m, chunk=c,
                             binning=binning)
        drop = torch.zeros(1, dtype=torch.int64, device="cuda")
        img = plan.dirty_image(uvw, vis, dropped=drop)
        st = plan.tile_stats()
        plan.reset()
        plan.grid(uvw[:m // 3], vis[:m // 3])
        plan.grid(uvw[m // 3:], vis[m // 3:])
        two = plan.new_image()
        plan.image_accumulate(two)
        out.append((img, two, st, int(drop.item())))
        plan.close()
    a, b = out
    tol = 1e-12 if precision == "fp64" else 1e-6
    for x in (a[0], a[1]):
        assert float(torch.linalg.vector_norm(x - b[0]) /
                     torch.linalg.vector_norm(b[0])) <= tol
    for key in ("busy", "idle", "strips", "record_reads"):
        assert a[2][key] == b[2][key], key
    assert a[3] == b[3]
    # Every dense tile is split, into no more items than there are slots.
    slots = 2 * m // chunk + 64
    assert a[2]["split"] == 4 * nw
    assert a[2]["extra_items"] + a[2]["split"] <= slots
