"""Sizes ws_grid_image_noalloc accepts and refuses, and dense tiles near its
limit.

The size test runs before anything touches a device: with a NULL image a
problem that fits gives WS_INVALID_ARG and one that does not
WS_WORKSPACE_TOO_SMALL, so the limits are checked here without a GPU.  Each
row holds the largest visibility count that fits.
"""
import ctypes as C
import math

import pytest

import paper_2301_06061_amd as ws
from paper_2301_06061_amd import _abi

LIMITS = [
    (dict(nu=512, nv=512, nw=8), 598_336),
    (dict(nu=512, nv=512, nw=8, precision="fp64"), 227_327),
    (dict(nu=1024, nv=1024, nw=6), 177_152),
    (dict(nu=1024, nv=1024, nw=3, precision="fp64"), 96_096),
    (dict(nu=128, nv=128, nw=4), 804_863),
    (dict(nu=128, nv=128, nw=4, precision="fp64", support=15), 482_739),
    (dict(nu=256, nv=128, nw=5, chunk=1024), 496_127),
    (dict(nu=512, nv=512, nw=8, tile=16), 730_186),
    (dict(nu=512, nv=256, nw=9, tile=32, binning="partition"), 829_920),
    (dict(nu=256, nv=256, nw=8, binning="hashed"), 1_263_637),
    (dict(nu=1024, nv=512, nw=15), 19_936),
    (dict(nu=64, nv=64, nw=1), 811_008),
    (dict(nu=2048, nv=2048, nw=1), 385_920),
    (dict(nu=512, nv=4096, nw=1), 493_493),
    (dict(nu=32, nv=16, nw=2, support=5), 1_028_266),
]


def _params(nu, nv, nw, support=7, precision="fp32", **kw):
    return ws.make_params(nu, nv, nw, 0.02, 0.02, -100.0, 100.0, support,
                          0.0, precision, **kw)


@pytest.mark.parametrize("kw,last", LIMITS)
def test_limits(kw, last):
    p = _params(**kw)

    def status(m):
        return _abi.lib().ws_grid_image_noalloc(
            C.byref(p), m, None, None, None, None, None, None)

    for m in (0, 1, last // 2, last - 1, last):
        assert status(m) == _abi.WS_INVALID_ARG, m
    for m in (last + 1, last + 1000, 2 * last, 50_000_000):
        assert status(m) == _abi.WS_WORKSPACE_TOO_SMALL, m


@pytest.mark.gpu
@pytest.mark.parametrize("precision,nw,m", [
    ("fp32", 6, 100_000), ("fp32", 6, 177_152), ("fp64", 3, 96_096)])
def test_dense_tile_near_the_limit(precision, nw, m):
    """Most visibilities in one tile of a stack that leaves little scratch
    for partial tiles: the image of the plan with caller buffers, in at
    most three times its time (the tile is split over many workgroups in
    both; one workgroup alone takes more than six times as long)."""
    torch = pytest.importorskip("torch")
    n = 1024
    fp64 = precision == "fp64"
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    f64 = dict(generator=g, device="cuda", dtype=torch.float64)
    uv = torch.rand(m, 2, **f64) * 40.0 + 10.0
    uv[::10] = (torch.rand(len(uv[::10]), 2, **f64) - 0.5) * (n - 10)
    w = torch.full((m, 1), -90.0, device="cuda", dtype=torch.float64)
    uvw = torch.cat([uv / 0.02, w], 1).contiguous()
    vis = torch.randn(m, generator=g, device="cuda",
                      dtype=torch.complex128 if fp64 else torch.complex64)
    p = _params(n, n, nw, precision=precision)
    plan = ws.WStackPlan(n, n, nw, 0.02, 0.02, -100.0, 100.0, 7,
                         precision=precision, max_vis=m)

    def timed(f):
        out, best = f(), math.inf
        for _ in range(5):
            a = torch.cuda.Event(enable_timing=True)
            b = torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return out, best

    got, t_got = timed(lambda: ws.api.grid_image_noalloc(p, uvw, vis, None))
    ref, t_ref = timed(lambda: plan.dirty_image(uvw, vis))
    plan.close()
    d, r = (got - ref).to(torch.complex128), ref.to(torch.complex128)
    if fp64:
        assert float(d.abs().max() / r.abs().max()) <= 1e-12
    else:
        assert float(torch.linalg.vector_norm(d) /
                     torch.linalg.vector_norm(r)) <= 1e-5
    assert t_got <= 3.0 * t_ref, (t_got, t_ref)


@pytest.mark.parametrize("m", [13, 30_000, 320_000])
def test_parameters_are_checked_once(m):
    """The checks of a plan with grid correction evaluate the kernel's
    transform a few hundred times, milliseconds of the host: the call does
    it once, also where it looks for a layout that fits."""
    import time
    p = _params(256, 256, 3, precision="fp64", kernel="es", correct=True)

    def best(f):
        times = []
        for _ in range(15):
            t = time.perf_counter()
            f()
            times.append(time.perf_counter() - t)
        return min(times)

    lib = _abi.lib()
    call = best(lambda: lib.ws_grid_image_noalloc(
        C.byref(p), m, None, None, None, None, None, None))
    check = best(lambda: lib.ws_validate_params(C.byref(p)))
    assert check > 1e-4
    assert call <= 1.5 * check, (call, check)
