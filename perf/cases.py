"""Workloads of the w-stacking library as its users run them.

Each case is one call sequence through the public Python entry points on
seeded inputs, from the smallest images, where launches and latency count,
to the largest grids:

  image     WStackPlan.dirty_image: one dirty image of flat visibilities
  noalloc   grid_image_noalloc: the same without a plan (serving, capture)
  slabs     baseline-major rows gridded in two additive slabs, then imaged
            (grid_rows twice + image_accumulate)
  rows      baseline-major rows through the one-call path (grid_image_rows)
  degrid    WStackPlan.degrid: model visibilities of a real image
  gradient  imaging_op forward and backward (degridding, then its adjoint)
  clean     MajorCycle.minor: one Hogbom minor cycle on the GPU
  batch     BatchedImager.run: many channels in one launch sequence

listed() gives the standing cases, draw() further ones of the same ranges,
prepare() the device inputs and the plan a program keeps, run() one pass,
work() the bytes and operations a pass cannot do without, exact() the same
outputs in 64-bit torch arithmetic.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2301_06061_amd as ws
from paper_2301_06061_amd.api import grid_image_noalloc, make_params
from paper_2301_06061_amd.autograd import imaging_op
from paper_2301_06061_amd.batch import BatchedImager
from paper_2301_06061_amd.clean import MajorCycle

C0 = 299_792_458.0  # m/s


def _case(kind, nu, nw, m, support=7, prec="fp32", law="core", fov=5.0,
          nv=0, weights=True, kernel="gauss", correct=False, **extra):
    c = {"kind": kind, "nu": nu, "nv": nv or nu, "nw": nw, "m": m,
         "support": support, "prec": prec, "law": law, "fov": fov,
         "weights": weights, "kernel": kernel, "correct": correct}
    c.update(extra)
    return c


def listed():
    def named(name, c):
        return dict(c, name=name)
    return [
        # A quick-look image of a short snapshot: latency and launches.
        named("image_128_fp32", _case("image", 128, 4, 20_000, fov=2.0)),
        # A serving loop without plans, unit weights, an odd count.
        named("noalloc_256_fp32", _case("noalloc", 256, 8, 30_011, fov=2.0,
                                        weights=False)),
        # Model prediction with the production kernel and its correction.
        named("degrid_256_es_fp64", _case("degrid", 256, 8, 50_021, fov=2.0,
                                          prec="fp64", law="gauss",
                                          kernel="es", correct=True)),
        # Plain w-stacking in the paper's precision.
        named("image_512_fp64", _case("image", 512, 8, 200_000, fov=1.0,
                                      prec="fp64", law="gauss")),
        # One channel of an ordinary observation.
        named("image_1024_fp32", _case("image", 1024, 16, 1_000_003)),
        # Baseline-major data arriving in slabs: additive gridding, 8
        # channels, four correlations combined into Stokes I.
        named("slabs_2048_fp32", _case("slabs", 2048, 16, 125_008, nchan=8,
                                       npol=4)),
        # A multi-channel observation: twelve channels in one sequence.
        named("batch_12ch_fp32", _case("batch", 1024, 16, 100_000,
                                       channels=12, m_hi=1_000_000,
                                       sizes=2)),
        # A minor cycle of the deconvolution at the headline image size.
        named("clean_4096_fp32", _case("clean", 4096, 1, 50_000, niter=200)),
        # The headline image: dense core, 1e7 visibilities, both precisions.
        named("image_4096_fp32", _case("image", 4096, 32, 10_000_000)),
        named("image_4096_fp64", _case("image", 4096, 32, 10_000_000,
                                       prec="fp64")),
        # Differentiable imaging: prediction and gradient.
        named("gradient_4096_fp32", _case("gradient", 4096, 32, 10_000_000,
                                          law="gauss", weights=False)),
        # A wide image beyond 4096 with a wider kernel.
        named("image_8192_k9_fp32", _case("image", 8192, 32, 20_000_007,
                                          support=9, fov=8.0)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["image", "image", "image", "noalloc", "slabs", "rows",
                       "degrid", "gradient", "clean", "batch"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    support = rng.choice([5, 7, 7, 9])
    law = rng.choice(["core", "gauss"])
    fov = rng.uniform(1.0, 6.0)
    kernel = rng.choice(["gauss", "gauss", "es"])
    correct = kernel == "es" and rng.random() < 0.5
    weights = rng.random() < 0.7
    if kind == "noalloc":
        n = 2 ** rng.randint(6, 8)
        return _case(kind, n, rng.randint(1, 6), _log_int(rng, 500, 60_000),
                     support, prec, law, fov, weights=weights, kernel=kernel,
                     correct=correct)
    if kind == "clean":
        return _case(kind, 2 ** rng.randint(8, 12), 1, 20_000, prec=prec,
                     fov=fov, niter=rng.randint(20, 200))
    if kind == "batch":
        return _case(kind, 512, 8, 20_000, support, "fp32", law, fov,
                     weights=weights, kernel=kernel, correct=correct,
                     channels=rng.randint(2, 12),
                     m_hi=_log_int(rng, 30_000, 600_000), sizes=3)
    # Grid edges from 64 to 8192, some of them not square.
    lu = rng.randint(6, 13 if kind == "image" else 12)
    lv = max(6, min(13, lu + rng.choice([-1, 0, 0, 0, 1])))
    nu, nv = 2 ** lu, 2 ** lv
    nw = rng.randint(1, 33)
    if prec == "fp64":
        nw = min(nw, max(1, 2 ** 29 // (nu * nv)))
    nw = min(nw, max(1, 2 ** 30 // (nu * nv)))
    m = _log_int(rng, 1_000, min(10_000_000, 8 * nu * nv + 10_000)) | 1
    extra = {}
    if kind in ("slabs", "rows"):
        extra = {"nchan": rng.randint(1, 9), "npol": rng.choice([1, 2, 4])}
        m = max(2, m // (extra["nchan"]))
    return _case(kind, nu, nw, m, support, prec, law, fov, nv=nv,
                 weights=weights, kernel=kernel, correct=correct, **extra)


# ---- inputs -----------------------------------------------------------------

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed, salt=0):
    g = torch.Generator(device=_dev())
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _coords(c, g, m, scale=1.0):
    """(u, v, w) in wavelengths and the plane range, on the GPU: a dense
    core (r = R U^2, w growing with r) or a Gaussian disk (uniform w)."""
    d, f64 = _dev(), torch.float64
    fov_l = math.radians(c["fov"])
    fov_m = fov_l * c["nv"] / c["nu"]
    n = min(c["nu"], c["nv"])
    half = (n / 2 - (c["support"] - 1) // 2 - 1) * scale
    wmax = (n / 2) / fov_l * scale
    th = torch.rand(m, generator=g, device=d, dtype=f64) * (2 * math.pi)
    t = torch.rand(m, generator=g, device=d, dtype=f64)
    if c["law"] == "core":
        r = half * t * t
        w = wmax * r / half + 0.1 * wmax * torch.randn(m, generator=g,
                                                       device=d, dtype=f64)
        lo, hi = float(w.min()), float(w.max())
        if not hi > lo:
            hi = lo + 1.0
    else:
        # Rayleigh radius cut at the disk's edge (inverse of its law).
        s = 0.25 * half
        cut = 1.0 - math.exp(-0.5 * (half / s) ** 2)
        r = s * torch.sqrt(-2.0 * torch.log1p(-t * cut))
        w = wmax * (2.0 * torch.rand(m, generator=g, device=d, dtype=f64) - 1)
        lo, hi = -wmax, wmax
    uvw = torch.stack([r * torch.cos(th) / fov_l, r * torch.sin(th) / fov_m,
                       w], dim=1).contiguous()
    return uvw, fov_l, fov_m, lo, hi


def _cplx(c):
    return torch.complex128 if c["prec"] == "fp64" else torch.complex64


def _noise(g, shape, dtype):
    return torch.randn(shape, generator=g, device=_dev(),
                       dtype=torch.float32).to(dtype) if not dtype.is_complex \
        else torch.randn(shape, generator=g, device=_dev(), dtype=dtype)


def _weights(c, g, shape):
    if not c["weights"]:
        return None
    return 0.5 + torch.rand(shape, generator=g, device=_dev(),
                            dtype=torch.float32)


def _flat(c, seed):
    """Flat visibilities of a case: uvw, vis, weight and the geometry."""
    g = _gen(seed)
    uvw, fov_l, fov_m, lo, hi = _coords(c, g, c["m"])
    vis = _noise(g, (c["m"],), _cplx(c))
    wt = _weights(c, g, (c["m"],))
    return SimpleNamespace(uvw=uvw, vis=vis, wt=wt, fov_l=fov_l, fov_m=fov_m,
                           lo=lo, hi=hi)


def _rows(c, seed):
    """Baseline-major rows: metres per row, channels over an octave."""
    g = _gen(seed)
    uvw, fov_l, fov_m, _, _ = _coords(c, g, c["m"])
    nch, npol = c["nchan"], c["npol"]
    freq = torch.linspace(100e6, 200e6, nch, device=_dev(),
                          dtype=torch.float64) if nch > 1 else \
        torch.full((1,), 200e6, device=_dev(), dtype=torch.float64)
    uvw_m = (uvw * (C0 / 200e6)).contiguous()
    wl = uvw_m[:, 2:3] * (freq / C0)
    lo, hi = float(wl.min()), float(wl.max())
    if not hi > lo:
        hi = lo + 1.0
    vis = _noise(g, (c["m"], nch, npol), _cplx(c))
    wt = _weights(c, g, (c["m"], npol))
    coeff = {1: [1.0], 2: [0.5, 0.5], 4: [0.5, 0.0, 0.0, 0.5]}[npol]
    return SimpleNamespace(uvw_m=uvw_m, freq=freq, vis=vis, wt=wt,
                           coeff=coeff, fov_l=fov_l, fov_m=fov_m, lo=lo,
                           hi=hi)


def _sky(c, seed):
    """A sparse real sky: 1000 point sources (fewer on small images)."""
    g = _gen(seed, 7)
    n = c["nu"] * c["nv"]
    k = min(1000, max(8, n // 64))
    idx = torch.unique(torch.randint(0, n, (k,), generator=g, device=_dev()))
    x = torch.zeros(n, device=_dev(), dtype=torch.float32)
    x[idx] = torch.randn(k, generator=g, device=_dev(),
                         dtype=torch.float32)[:idx.numel()]
    rd = torch.float64 if c["prec"] == "fp64" else torch.float32
    return x.reshape(c["nv"], c["nu"]).to(rd)


def _clean_images(c, seed):
    """Dirty beam and residual of point sources, from a sampled uv plane."""
    g = _gen(seed)
    d, n, nv = _dev(), c["nu"], c["nv"]
    uvw, *_ = _coords(dict(c, support=7), g, c["m"])
    fov = math.radians(c["fov"])
    i = torch.floor(uvw[:, 0] * fov + n / 2 + 0.5).long().clamp(1, n - 1)
    j = torch.floor(uvw[:, 1] * fov * nv / n + nv / 2 + 0.5).long().clamp(
        1, nv - 1)
    s = torch.zeros(nv, n, device=d, dtype=torch.float64)
    s.view(-1)[j * n + i] = 1.0  # uniform weighting of the sampled cells
    s.view(-1)[(nv - j) * n + (n - i)] = 1.0
    s = torch.fft.ifftshift(s)
    psf = torch.fft.fft2(s).real / s.sum()
    src = torch.zeros(nv * n, device=d, dtype=torch.float64)
    k = 40
    idx = torch.randint(0, nv * n, (k,), generator=g, device=d)
    idx = torch.unique(idx)
    src[idx] = 1.0 + 9.0 * torch.rand(k, generator=g, device=d,
                                      dtype=torch.float64)[:idx.numel()]
    dirty = torch.fft.ifft2(torch.fft.fft2(src.reshape(nv, n)) *
                            torch.fft.fft2(psf)).real
    noise = torch.randn(nv, n, generator=g, device=d, dtype=torch.float64)
    dirty = dirty + 0.02 * noise
    rd = torch.float64 if c["prec"] == "fp64" else torch.float32
    return torch.fft.fftshift(psf).to(rd).contiguous(), dirty.to(rd)


def _channels(c, seed):
    """Per-channel geometry (from the case alone) and data (from the seed)."""
    rng = np.random.default_rng(c["channels"] * 1000 + c["sizes"])
    out = []
    for i in range(c["channels"]):
        n = c["nu"] * int(2 ** rng.integers(0, c["sizes"]))
        m = int(round(math.exp(rng.uniform(math.log(c["m"]),
                                           math.log(c["m_hi"])))))
        cc = dict(c, nu=n, nv=n, m=m)
        scale = 0.5 + 0.5 * i / max(1, c["channels"] - 1)
        g = _gen(seed, 100 + i)
        uvw, fov_l, fov_m, lo, hi = _coords(cc, g, m, scale)
        vis = _noise(g, (m,), _cplx(c))
        out.append((cc, SimpleNamespace(uvw=uvw, vis=vis,
                                        wt=_weights(c, g, (m,)),
                                        fov_l=fov_l, fov_m=fov_m, lo=lo,
                                        hi=hi)))
    return out


def _plan(c, d, m):
    return ws.WStackPlan(c["nu"], c["nv"], c["nw"], d.fov_l, d.fov_m, d.lo,
                         d.hi, c["support"], precision=c["prec"], max_vis=m,
                         kernel=c["kernel"], correct=c["correct"])


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "clean":
        beam, dirty = _clean_images(c, seed)
        plan = ws.WStackPlan(c["nu"], c["nv"], 1, math.radians(c["fov"]),
                             math.radians(c["fov"]) * c["nv"] / c["nu"],
                             -1.0, 1.0, precision=c["prec"], max_vis=1)
        mc = MajorCycle(plan, torch.zeros(1, 3, device=_dev(),
                                          dtype=torch.float64),
                        torch.ones(1, device=_dev(), dtype=_cplx(c)))
        mc.beam.copy_(beam)
        picks = torch.full((c["niter"],), -1, dtype=torch.int32,
                           device=_dev())
        return SimpleNamespace(c=c, mc=mc, dirty=dirty, picks=picks)
    if kind == "batch":
        chans = _channels(c, seed)
        loads = [SimpleNamespace(nu=cc["nu"], nv=cc["nv"], nw=cc["nw"],
                                 fov_l=d.fov_l, fov_m=d.fov_m, w_min=d.lo,
                                 w_max=d.hi, support=cc["support"],
                                 kernel=cc["kernel"], correct=cc["correct"])
                 for cc, d in chans]
        b = BatchedImager(loads, [d.uvw for _, d in chans],
                          [d.vis for _, d in chans],
                          [d.wt for _, d in chans], precision=c["prec"])
        return SimpleNamespace(c=c, batch=b)
    if kind in ("slabs", "rows"):
        d = _rows(c, seed)
        if kind == "rows":
            return SimpleNamespace(c=c, d=d,
                                   plan=_plan(c, d, c["m"] * c["nchan"]))
        cut = c["m"] // 2
        parts = [(d.uvw_m[:cut], d.vis[:cut],
                  None if d.wt is None else d.wt[:cut]),
                 (d.uvw_m[cut:], d.vis[cut:],
                  None if d.wt is None else d.wt[cut:])]
        return SimpleNamespace(c=c, d=d, parts=parts,
                               plan=_plan(c, d, (c["m"] - cut) * c["nchan"]))
    d = _flat(c, seed)
    if kind == "noalloc":
        p = make_params(c["nu"], c["nv"], c["nw"], d.fov_l, d.fov_m, d.lo,
                        d.hi, c["support"], precision=c["prec"],
                        kernel=c["kernel"], correct=c["correct"])
        return SimpleNamespace(c=c, d=d, params=p)
    s = SimpleNamespace(c=c, d=d, plan=_plan(c, d, c["m"]))
    if kind in ("degrid", "gradient"):
        s.x = _sky(c, seed)
        d.vis_grad, d.vis = d.vis, None
    return s


def run(state):
    kind, c = state.c["kind"], state.c
    if kind == "image":
        d = state.d
        return state.plan.dirty_image(d.uvw, d.vis, d.wt)
    if kind == "noalloc":
        d = state.d
        return grid_image_noalloc(state.params, d.uvw, d.vis, d.wt)
    if kind == "rows":
        d = state.d
        return state.plan.grid_image_rows(d.uvw_m, d.freq, d.vis, d.wt,
                                          d.coeff)
    if kind == "slabs":
        state.plan.reset()
        for uvw_m, vis, wt in state.parts:
            state.plan.grid_rows(uvw_m, state.d.freq, vis, wt, state.d.coeff)
        img = state.plan.new_image()
        state.plan.image_accumulate(img)
        return img
    if kind == "degrid":
        return state.plan.degrid(state.x, state.d.uvw, state.d.wt)
    if kind == "gradient":
        x = state.x.detach().requires_grad_(True)
        y = imaging_op(x, state.plan, state.d.uvw, state.d.wt)
        (gx,) = torch.autograd.grad(y, x, state.d.vis_grad)
        return {"vis": y.detach(), "grad": gx}
    if kind == "clean":
        mc = state.mc
        mc.residual.copy_(state.dirty)
        mc.model.zero_()
        mc.minor(c["niter"], 0.1, 0.0, state.picks)
        return {"residual": mc.residual, "model": mc.model,
                "picks": state.picks}
    return state.batch.run()


# ---- work -------------------------------------------------------------------

def _image_work(c, m, in_bytes, passes=1):
    cells, e = c["nu"] * c["nv"], 16 if c["prec"] == "fp64" else 8
    fl = m * (4.0 * c["support"] ** 2) + c["nw"] * cells * (
        5.0 * math.log2(cells) + 8.0)
    return {"bytes": float(in_bytes + passes * cells * e),
            "flops": passes * fl}


def work(case):
    c, kind = case, case["kind"]
    cells = c["nu"] * c["nv"]
    e = 16 if c["prec"] == "fp64" else 8
    per = 24 + e + (4 if c["weights"] else 0)
    if kind == "clean":
        # Residual, beam and model once; two operations a pixel and step.
        return {"bytes": 5.0 * cells * e / 2, "flops": 2.0 * cells *
                c["niter"]}
    if kind == "batch":
        rng = np.random.default_rng(c["channels"] * 1000 + c["sizes"])
        tot = {"bytes": 0.0, "flops": 0.0}
        for _ in range(c["channels"]):
            n = c["nu"] * int(2 ** rng.integers(0, c["sizes"]))
            m = int(round(math.exp(rng.uniform(math.log(c["m"]),
                                               math.log(c["m_hi"])))))
            w = _image_work(dict(c, nu=n, nv=n), m, m * per)
            tot = {k: tot[k] + w[k] for k in tot}
        return tot
    if kind in ("slabs", "rows"):
        m = c["m"] * c["nchan"]
        row = 24 + (4 * c["npol"] if c["weights"] else 0)
        return _image_work(c, m, c["m"] * row + m * c["npol"] * e)
    if kind == "degrid":
        w = _image_work(c, c["m"], c["m"] * per)
        return {"bytes": w["bytes"] - cells * e / 2, "flops": w["flops"]}
    if kind == "gradient":
        w = _image_work(c, c["m"], c["m"] * per, 2)
        return {"bytes": w["bytes"] + c["m"] * e - cells * e,
                "flops": w["flops"]}
    return _image_work(c, c["m"], c["m"] * per)


# ---- 64-bit values ----------------------------------------------------------

def _phi(c, d):
    """1-D kernel factor at offsets d (cells) and the 2-D norm."""
    K = c["support"]
    if c["kernel"] == "es":
        z = 2.0 * d / K
        return torch.exp(2.3 * K * (torch.sqrt(torch.clamp(1 - z * z, min=0))
                                    - 1.0))
    s = K / 7.0
    return torch.exp(-d * d / (2.0 * s * s))


def _psi(c, f):
    """Transform of the 1-D kernel truncated to its support at f (numpy)."""
    K = c["support"]
    x, w = np.polynomial.legendre.leggauss(160)
    f = np.asarray(f, dtype=np.float64)
    if c["kernel"] == "es":
        t = x * (math.pi / 2)
        d, g = K / 2 * np.sin(t), np.exp(2.3 * K * (np.cos(t) - 1.0))
        w = w * (math.pi / 2) * (K / 2) * np.cos(t)
    else:
        d = K / 2 * x
        g = np.exp(-d * d / (2.0 * (K / 7.0) ** 2))
        w = w * (K / 2)
    return np.cos(2 * math.pi * np.multiply.outer(f, d)) @ (w * g)


def _norm(c):
    if c["kernel"] == "es":
        return 1.0 / float(_psi(c, 0.0)) ** 2
    return 1.0 / (2.0 * math.pi * (c["support"] / 7.0) ** 2)


def _taps(c, uvw, d):
    """Flat cell index, weight and on-grid mask of every tap, and planes."""
    K, h = c["support"], (c["support"] - 1) // 2
    x = uvw[:, 0] * d.fov_l + 0.5 * c["nu"]
    y = uvw[:, 1] * d.fov_m + 0.5 * c["nv"]
    i0, j0 = torch.floor(x + 0.5), torch.floor(y + 0.5)
    a = torch.arange(-h, h + 1, device=uvw.device, dtype=torch.float64)
    gx = _phi(c, (i0 - x)[:, None] + a)
    gy = _phi(c, (j0 - y)[:, None] + a)
    ii, jj = (i0[:, None] + a).long(), (j0[:, None] + a).long()
    on = (((ii >= 0) & (ii < c["nu"]))[:, None, :] &
          ((jj >= 0) & (jj < c["nv"]))[:, :, None])
    idx = jj[:, :, None] * c["nu"] + ii[:, None, :]
    wt = (gy[:, :, None] * gx[:, None, :]) * on
    return torch.where(on, idx, torch.zeros_like(idx)), wt


def _plane(c, uvw, d):
    if c["nw"] == 1:
        return torch.zeros(uvw.shape[0], dtype=torch.long, device=uvw.device)
    dw = (d.hi - d.lo) / c["nw"]
    return torch.floor((uvw[:, 2] - d.lo) / dw).clamp(0, c["nw"] - 1).long()


def _w_centre(c, d, k):
    if c["nw"] == 1:
        return 0.5 * (d.lo + d.hi)
    return d.lo + (k + 0.5) * (d.hi - d.lo) / c["nw"]


def _nm1(c, d):
    f64, dev = torch.float64, _dev()
    l = (torch.arange(c["nu"], device=dev, dtype=f64) - c["nu"] // 2) * (
        d.fov_l / c["nu"])
    m = (torch.arange(c["nv"], device=dev, dtype=f64) - c["nv"] // 2) * (
        d.fov_m / c["nv"])
    r2 = m[:, None] ** 2 + l[None, :] ** 2
    return -r2 / (1.0 + torch.sqrt(1.0 - r2))


def _screen(nm1, w):
    t = w * nm1
    t = (t - torch.round(t)) * (2 * math.pi)
    return torch.polar(torch.ones_like(t), t)


def _correction(c):
    fu = (np.arange(c["nu"]) - c["nu"] // 2) / c["nu"]
    fv = (np.arange(c["nv"]) - c["nv"] // 2) / c["nv"]
    cu = torch.from_numpy(1.0 / (_norm(c) * _psi(c, fu))).to(_dev())
    cv = torch.from_numpy(1.0 / _psi(c, fv)).to(_dev())
    return cv[:, None] * cu[None, :]


_CHUNK = 1 << 19


def _exact_image(c, d, uvw, val):
    """Dirty image of values `val` (weights applied) in complex128."""
    cells, cn = c["nu"] * c["nv"], _norm(c)
    order = torch.argsort(_plane(c, uvw, d))
    counts = torch.bincount(_plane(c, uvw, d), minlength=c["nw"]).tolist()
    nm1 = _nm1(c, d)
    img = torch.zeros(c["nv"], c["nu"], dtype=torch.complex128, device=_dev())
    at = 0
    for k in range(c["nw"]):
        sel, at = order[at:at + counts[k]], at + counts[k]
        if counts[k] == 0:
            continue
        P = torch.zeros(cells, 2, dtype=torch.float64, device=_dev())
        for b in range(0, counts[k], _CHUNK):
            s = sel[b:b + _CHUNK]
            idx, wt = _taps(c, uvw[s], d)
            v = torch.view_as_real(val[s].to(torch.complex128)) * cn
            P.index_add_(0, idx.reshape(-1),
                         (wt[..., None] * v[:, None, None, :]).reshape(-1, 2))
        F = torch.fft.ifftshift(torch.view_as_complex(P).reshape(c["nv"],
                                                                 c["nu"]))
        del P
        F = torch.fft.fftshift(torch.fft.ifft2(F, norm="forward"))
        img += F * _screen(nm1, _w_centre(c, d, k))
    return img * _correction(c) if c["correct"] else img


def _exact_degrid(c, d, x):
    """Visibilities of a real image in complex128."""
    X = x.to(torch.complex128)
    if c["correct"]:
        X = X * _correction(c)
    nm1, cn = _nm1(c, d), _norm(c)
    pl = _plane(c, d.uvw, d)
    order = torch.argsort(pl)
    counts = torch.bincount(pl, minlength=c["nw"]).tolist()
    out = torch.zeros(c["m"], dtype=torch.complex128, device=_dev())
    at = 0
    for k in range(c["nw"]):
        sel, at = order[at:at + counts[k]], at + counts[k]
        if counts[k] == 0:
            continue
        F = torch.fft.ifftshift(X * _screen(nm1, _w_centre(c, d, k)).conj())
        Q = torch.view_as_real(torch.fft.fftshift(torch.fft.fft2(F)).reshape(
            -1).contiguous())
        for b in range(0, counts[k], _CHUNK):
            s = sel[b:b + _CHUNK]
            idx, wt = _taps(c, d.uvw[s], d)
            v = (Q[idx] * wt[..., None]).sum(dim=(1, 2)) * cn
            out[s] = torch.view_as_complex(v.contiguous())
    return out if d.wt is None else out * d.wt.to(torch.float64)


def _exact_clean(c, seed):
    beam, d = _clean_images(c, seed)
    beam, d = beam.to(torch.float64), d.to(torch.float64).clone()
    nv, nu = c["nv"], c["nu"]
    model = torch.zeros_like(d)
    flat = d.view(-1)
    for _ in range(c["niter"]):
        idx = int(torch.argmax(flat.abs()))
        q, p = idx // nu, idx % nu
        a = 0.1 * float(flat[idx])
        model[q, p] += a
        q0, p0 = max(0, q - nv // 2), max(0, p - nu // 2)
        q1, p1 = min(nv, q + nv - nv // 2), min(nu, p + nu - nu // 2)
        d[q0:q1, p0:p1] -= a * beam[q0 - q + nv // 2:q1 - q + nv // 2,
                                    p0 - p + nu // 2:p1 - p + nu // 2]
    return {"residual": d, "model": model, "picks": None}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "clean":
        return _exact_clean(c, seed)
    if kind == "batch":
        return [_exact_image(cc, d, d.uvw,
                             d.vis if d.wt is None else
                             d.vis.to(torch.complex128) * d.wt)
                for cc, d in _channels(c, seed)]
    if kind in ("slabs", "rows"):
        d = _rows(c, seed)
        v = d.vis.to(torch.complex128)
        if d.wt is not None:
            v = v * d.wt.to(torch.float64)[:, None, :]
        co = torch.tensor(d.coeff, dtype=torch.complex128, device=_dev())
        val = (v * co).sum(dim=2).reshape(-1)
        uvw = (d.uvw_m[:, None, :] * (d.freq / C0)[None, :, None]).reshape(
            -1, 3)
        return _exact_image(c, d, uvw, val)
    d = _flat(c, seed)
    val = d.vis.to(torch.complex128)
    if d.wt is not None:
        val = val * d.wt.to(torch.float64)
    if kind == "degrid":
        return _exact_degrid(c, d, _sky(c, seed))
    if kind == "gradient":
        return {"vis": _exact_degrid(c, d, _sky(c, seed)),
                "grad": _exact_image(c, d, d.uvw, val).real.contiguous()}
    return _exact_image(c, d, d.uvw, val)
