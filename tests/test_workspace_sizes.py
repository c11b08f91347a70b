"""Workspace of automatic work items: the scratch for the partial tiles of
split tiles stays within its bound, and a batch's plans reserve what the
batch's items need."""
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

    # Slots of 64 KB: twice the visibilities and 64 over (up to 16384 keys,
    # nine a tile, and 2^20 visibilities); else 2^18 records over, or all that
    # four reads of each can need.
    tiles = (n // 64) ** 2 * nw

    def slots(c):
        four = 4 * m // c
        if 9 * tiles <= 16384 and m <= 2 ** 20:
            return 2 * m // c + 64
        return max(1, min(2 * m // c + 2 ** 18 // c, four + min(four, tiles)))

    # The least power of two from 512 to 4096 that reaches the square root of
    # m and whose slots stay within the bound.
    c = 512
    while c < 4096 and (c * c < m or slots(c) > 4096 or
                        slots(c) * 65536 > max(160 * MIB, planes // 16)):
        c *= 2
    # A plan that asks for c has 64 slots over: the workspaces differ by the
    # slots (and up to 100 bytes of descriptor and list entry for each).
    more = min(4096, slots(c)) - min(4096, 2 * m // c + 64)
    diff = auto - _bytes(n, nw, m, precision, chunk=c)[1]
    ends = sorted([more * 65536, more * 65636])
    assert ends[0] - 1024 <= diff <= ends[1] + 1024, (c, more, diff)


@pytest.mark.gpu
def test_batch_plans_reserve_for_the_batch():
    torch = pytest.importorskip("torch")
    from types import SimpleNamespace
    from paper_2301_06061_amd.batch import BatchedImager
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    n, nw, fov = 128, 2, 0.02
    wl = SimpleNamespace(nu=n, nv=n, nw=nw, fov_l=fov, fov_m=fov, w_min=-1.0,
                         w_max=1.0, support=7, sigma=0.0)

    def data(m):
        f64 = dict(generator=g, device="cuda", dtype=torch.float64)
        uv = (torch.rand(m, 2, **f64) - 0.5) * (n - 10) / fov
        return (torch.cat([uv, torch.rand(m, 1, **f64) * 2 - 1],
                          1).contiguous(),
                torch.randn(m, generator=g, device="cuda",
                            dtype=torch.complex64))

    # 4.3e6 visibilities together: items of 4096, whatever a plan's own.
    for counts, params, chunks in (
            ([2_200_000, 2_000_000, 100_000], None, [4096] * 3),
            ([2_200_000, 2_000_000, 100_000],
             [(0, 0), (32, 0), (0, 2048)], [4096, 4096, 2048]),
            ([200_000, 100_000], None, [0, 0])):
        uvw, vis = zip(*[data(m) for m in counts])
        b = BatchedImager([wl] * len(counts), uvw, vis, precision="fp32",
                          params=params)
        assert b.tuned == (params or [(0, 0)] * len(counts))
        images = [t.clone() for t in b.run()]
        for i, (p, m) in enumerate(zip(b.plans, counts)):
            q = ws.make_params(n, n, nw, fov, fov, -1.0, 1.0, 7, 0.0, "fp32",
                               tile=b.tuned[i][0], chunk=chunks[i])
            assert p.work.numel() == ws.workspace_bytes(q, m)[1], i
            plan = ws.WStackPlan(n, n, nw, fov, fov, -1.0, 1.0, 7, max_vis=m)
            ref = plan.dirty_image(uvw[i], vis[i])
            err = float(torch.linalg.vector_norm(images[i] - ref) /
                        torch.linalg.vector_norm(ref))
            assert err <= 1e-6, (i, err)
            plan.close()
        b.close()
