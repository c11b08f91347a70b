"""Row-transform twiddles of the fused row kernels are the plan's table
entries, each rounded once.

One impulse in a row meets no rounding at all in the stages that take it as
input 0 of their butterflies, and one product with a twiddle in the stage that
takes it as input r.  A visibility of value 1 on cell (e, 0) of the only plane
(K = 1, w = 0: no screen, a column transform of ones) therefore images to
(-1)^(e + p + q) W_N^(e p), and at the pixels p where stage P's output index is
0 the number is that twiddle itself.  FP32: equal to the rounded cosine and
sine, bit for bit.  FP64: equal, bit for bit, to the same table entry met
through r = 1.  Degridding likewise, from an image of one pixel.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2301_06061_amd as ws  # noqa: E402

pytestmark = pytest.mark.gpu
NV = 64


def _stages(n):
    """(NS, RAD) of every stage after the first: radix 8, the rest last."""
    out, ns = [], 1
    while ns < n:
        rad = min(8, n // ns)
        if ns > 1:
            out.append((ns, rad))
        ns *= rad
    return out


def _probes(n):
    """(e, pixels) of every twiddle input of every stage."""
    for ns, rad in _stages(n):
        for r in range(1, rad):
            p = np.arange(n)
            yield r * n // (ns * rad), p[p % (ns * rad) < ns]


def _plan(n, precision, m):
    fov = 2.0 ** -7  # cell coordinates u * fov + n / 2 are exact
    return ws.WStackPlan(n, NV, 1, fov, fov, 0.0, 0.0, 1,
                         1.0 / np.sqrt(2.0 * np.pi),  # c = 1
                         precision, max_vis=m), fov


def _cells(n, i, fov):
    uvw = np.zeros((len(i), 3))
    uvw[:, 0] = (np.asarray(i) - n // 2) / fov
    uvw[:, 1] = (0 - NV // 2) / fov
    return torch.from_numpy(uvw).cuda()


def _exact(n):
    a = np.exp(2j * np.pi * np.arange(n) / n)
    re, im = a.real.copy(), a.imag.copy()
    re[np.abs(re) < 1e-12] = 0.0
    im[np.abs(im) < 1e-12] = 0.0
    return re + 1j * im


def _check(n, precision, seen):
    """seen: (twiddle index, value) arrays, one per probe."""
    idx = np.concatenate([a for a, _ in seen])
    val = np.concatenate([b for _, b in seen])
    if precision == "fp32":
        assert np.array_equal(val, _exact(n)[idx].astype(np.complex64))
        return
    assert np.abs(val - _exact(n)[idx]).max() <= 1e-14
    # r = 1 of the last stage: entries 0 .. NS-1.
    ns, rad = _stages(n)[-1]
    first = seen[-(rad - 1)]
    ref = np.full(n, np.nan + 0j)
    ref[first[0]] = first[1]
    known = idx < ns
    assert np.array_equal(val[known], ref[idx[known]])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [32, 64, 256, 512, 1024, 2048, 4096])
def test_imaging_rows_use_table_entries(n, precision):
    plan, fov = _plan(n, precision, 1)
    one = torch.ones(1, dtype=plan.cdtype, device="cuda")
    seen = []
    for e, p in _probes(n):
        img = plan.dirty_image(_cells(n, [e], fov), one).cpu().numpy()
        for q in (0, 1, NV - 1):
            sign = 1.0 - 2.0 * ((e + p + q) & 1)
            seen.append(((e * p) % n, img[q, p] * sign.astype(img.real.dtype)))
    plan.close()
    _check(n, precision, seen[2::3])
    for a, b in zip(seen[0::3], seen[1::3]):
        assert np.array_equal(a[1], b[1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [32, 64, 256, 512, 1024, 2048, 4096])
def test_degridding_rows_use_table_entries(n, precision):
    plan, fov = _plan(n, precision, n)
    uvw = _cells(n, np.arange(n), fov)
    x = torch.zeros((NV, n), dtype=plan.rdtype, device="cuda")
    seen = []
    for e, p in _probes(n):
        x.zero_()
        x[0, e] = 1.0
        vis = plan.degrid(x, uvw).cpu().numpy()
        sign = (1.0 - 2.0 * ((e + p) & 1)).astype(vis.real.dtype)
        seen.append(((e * p) % n, np.conj(vis[p]) * sign))
    plan.close()
    _check(n, precision, seen)
