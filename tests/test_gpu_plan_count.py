"""Capacity planning counts the visible pairs and the instances without
sorting: the same numbers as the binning that follows, at the edges of its
blocks (8192 pairs) and for both projection kernels, surfels and 3D
Gaussians."""
import math

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import scenes
from paper_2501_08174_amd.raster import Params, Pruner3D, Rasterizer, ViewBatch

pytestmark = pytest.mark.gpu


def _views(V):
    cams = []
    for v in range(V):
        c = np.array([math.cos(v), math.sin(v), 0.3 * v - 0.2]) * 3.0
        cams.append(scenes.make_camera(scenes.look_at_rotation(c), c, 150 + 40 * v, 90 + 60 * v))
    return ViewBatch(cams)


def _arrays(N):
    g = torch.Generator(device="cuda").manual_seed(N)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")
    # a wider cloud than the views see, some too transparent: culled pairs among the others
    return (r(N, 3) * 6.0 - 3.0, torch.exp(math.log(0.005) + r(N, 2) * math.log(40.0)),
            torch.randn(N, 4, generator=g, device="cuda"), r(N), torch.zeros(N, 1, 3, device="cuda"))


@pytest.mark.parametrize("N,V", [(1, 1), (8191, 1), (8192, 1), (8193, 1), (2731, 3), (4097, 4), (200_000, 2)])
def test_counts_match_the_binning(N, V):
    views = _views(V)
    m, s, q, o, sh = _arrays(N)
    r = Rasterizer(N, views, 0)
    need = r.plan_capacity(Params(m, s, q, o, sh))
    planned = r.counters.cpu().numpy().view(np.uint32)[:2].copy()
    r.bin()
    vis, got, stored, status = r.status()
    assert (planned[0], planned[1]) == (vis, got) and need == got and stored == got and status == 0
    p3 = Pruner3D(N, views)
    args = (m, torch.cat([s, s[:, :1]], dim=1).contiguous(), q, o)
    need = p3.plan_capacity(*args)
    planned = p3.counters.cpu().numpy().view(np.uint32)[:2].copy()
    p3.bin()
    vis, got, stored, status = p3.status()
    assert (planned[0], planned[1]) == (vis, got) and need == got and stored == got and status == 0
