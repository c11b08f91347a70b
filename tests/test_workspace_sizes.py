"""Workspace of automatic work items: the scratch for the partial tiles of
split tiles stays within its bound, and a batch's plans reserve what the
batch's items need."""
import math

import numpy as np
import pytest

import paper_2301_06061_amd as ws

MIB = 1 << 20


def _bytes(n, nw, m, precision="fp32", **kw):
    p = ws.make_params(n, n, nw, 0.02, 0.02, -100.0, 100.0, 7, 0.0, precision,
                       **kw)
    return ws.workspace_bytes(p, m)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,nw", [(64, 1), (512, 4), (1024, 16), (2048, 32),
                                  (4096, 32)])
@pytest.mark.parametrize("m", [1, 20_000, 262_144, 262_145, 1_000_000,
                               2_031_616, 2_031_617, 4_000_000, 4_194_304,
                               10_000_000])
def test_partial_tiles_stay_within_their_bound(n, nw, m, precision):
    planes, auto = _bytes(n, nw, m, precision)
    sizes = {c: _bytes(n, nw, m, precision, chunk=c)[1]
             for c in (512, 1024, 2048, 4096)}
    least = min(4096, max(512, 2 ** math.ceil(math.log2(m) / 2)))
    # (a few visibilities take the same workspace with any of them)
    used = [c for c in sizes if c >= least and sizes[c] == auto]
    assert used, "automatic items are one of the four sizes"
    c = used[0]

    def partials(c):
        return min(4096, 2 * m // c + 64) * 64 * 64 * 16

    bound = max(128 * MIB, planes // 16)
    if c < 4096:
        assert partials(c) <= bound
    if c > least:  # only as large as the bound asks for
        assert partials(c // 2) > bound


@pytest.mark.gpu
def test_batch_plans_reserve_for_the_batch():
    torch = pytest.importorskip("torch")
    import synth
    from oracle import wstack as o
    from paper_2301_06061_amd.batch import BatchedImager
    wls = [synth.random_case(90 + i, n=n, nw=2, support=7, m=m, law="core",
                             precision=0)
           for i, (n, m) in enumerate([(128, 150_000), (64, 100_000),
                                       (128, 20_000)])]
    dev = [[torch.from_numpy(np.ascontiguousarray(getattr(w, k))).cuda()
            for w in wls] for k in ("uvw", "vis", "weight")]
    for params, chunks in ((None, [1024] * 3),
                           ([(0, 0), (32, 0), (0, 2048)], [1024, 1024, 2048])):
        b = BatchedImager(wls, *dev, precision="fp32", params=params)
        assert b.tuned == (params or [(0, 0)] * 3)
        for i, (w, p) in enumerate(zip(wls, b.plans)):
            q = ws.make_params(w.nu, w.nv, w.nw, w.fov_l, w.fov_m, w.w_min,
                               w.w_max, w.support, w.sigma, "fp32",
                               tile=b.tuned[i][0], chunk=chunks[i])
            assert p.work.numel() == ws.workspace_bytes(q, w.m)[1], i
        for w, img in zip(wls, b.run()):
            ref = o.image(o.Params.of(w), w.uvw, w.vis, w.weight)
            err = np.linalg.norm(img.cpu().numpy() - ref)
            assert err <= 1e-5 * np.linalg.norm(ref)
        b.close()
