"""The 2DGS regularisers at the edges of the 32x16 tiles and of the halos,
against the FP64 oracle, and with infinite depths."""
import numpy as np
import pytest
import torch

import oracle
from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import RegularizerLoss, ViewBatch

pytestmark = pytest.mark.gpu


def _run(sizes, spoil=None, median=False):
    cams = [scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -4.0]), W, H) for W, H in sizes]
    views = ViewBatch(cams)
    g = torch.Generator(device="cuda").manual_seed(views.P)
    rand = lambda n: torch.rand(n, generator=g, device="cuda")
    alpha = 0.3 + 0.7 * rand(views.P)
    depth = alpha * (3.0 + 0.5 * rand(views.P))
    if spoil:
        spoil(alpha, depth)
    maps = [alpha, depth, rand(3 * views.P) - 0.5, 0.05 * rand(views.P)] + ([3.0 + 0.5 * rand(views.P)] if median else [])
    maps = [m.requires_grad_(True) for m in maps]
    ws = torch.zeros(_lib.workspace_bytes_loss(views.V, views.host), dtype=torch.uint8, device="cuda")
    total, per = RegularizerLoss.apply(*maps[:4], views, 100.0, 0.05, ws, *maps[4:])
    total.backward()
    return cams, views, maps, total, per


@pytest.mark.parametrize("sizes", [[(1, 1)], [(3, 3)], [(32, 16)], [(33, 17), (31, 15)], [(64, 33), (5, 70), (97, 1)],
                                   [(35, 18)] * 9])
def test_edges_of_tiles(sizes):
    cams, views, maps, total, per = _run(sizes)
    cut = lambda m, k=1: [m.detach().cpu().numpy()[views.view_slice(v, k)].reshape((k,) * (k > 1) + (H, W))
                          for v, (W, H) in enumerate(sizes)]
    ref = oracle.regularizer_loss64(cut(maps[0]), cut(maps[1]), cut(maps[2], 3), cut(maps[3]), cams, 100.0, 0.05)
    # means of values of order one: a few eps; the gradients are differences
    # of quotients by a normal's length, some hundred eps of the largest
    assert abs(float(total.detach()) - ref["total"]) <= 1e-5 * abs(ref["total"]) + 1e-6
    for v in range(views.V):
        for k, (m, n) in {"alpha": (0, 1), "depth": (1, 1), "normal": (2, 3), "dist": (3, 1)}.items():
            got, want = maps[m].grad.cpu().numpy()[views.view_slice(v, n)], ref["grads"][v][k].reshape(-1)
            assert np.abs(got - want).max() <= 2e-4 * max(np.abs(want).max(), 1e-30), (v, k)


def test_infinite_and_empty_pixels():
    """An infinite point spoils its neighbours' normals and nothing beyond
    their own neighbours; a normal of overflowing length is zero."""
    def spoil(alpha, depth):
        depth[20 * 64 + 40] = float("inf")
        alpha[5 * 64 + 5] = 0.0
        depth[30 * 64 + 10] = 1e25

    _, _, maps, _, _ = _run([(64, 40)], spoil)
    bad = ~torch.isfinite(maps[2].grad.view(3, 40, 64)).all(0)
    assert set(map(tuple, bad.nonzero().tolist())) <= {(20, 39), (20, 41), (19, 40), (21, 40)}
    assert bool(bad.any())
    assert torch.isfinite(maps[2].grad.view(3, 40, 64)[:, 29:32, 9:12]).all()
    assert float(maps[1].grad[5 * 64 + 5]) == 0.0
