"""Compositing with the entries' records read through the scalar cache (many
tiles) and as broadcasts from LDS (few): a small view gives the same images
and decisions, bit for bit, alone and beside a frame that brings the batch over
the limit, and the same record gradients up to the order of their sums."""
import math

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import scenes
from paper_2501_08174_amd.raster import Params, Rasterizer, ViewBatch

pytestmark = pytest.mark.gpu

N = 900
SMALL, LARGE = (75, 53), (1640, 1290)          # 2.1 million pixels: beyond the limit of either kernel


def _params(seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")
    return Params(r(N, 3) * 2.0 - 1.0, torch.exp(math.log(0.02) + r(N, 2) * math.log(20.0)),
                  torch.randn(N, 4, generator=g, device="cuda"), torch.clamp(r(N), 0.02, 0.99),
                  torch.randn(N, 4, 3, generator=g, device="cuda") * 0.3)


def _camera(direction, size):
    c = np.asarray(direction, np.float64)
    c *= 4.0 / np.linalg.norm(c)
    return scenes.make_camera(scenes.look_at_rotation(c), c, *size)


def _run(cams, tile, kind, p):
    views = ViewBatch(cams, tile=tile)
    r = Rasterizer(N, views, 1)
    r.plan_capacity(p)
    g = torch.Generator(device="cuda").manual_seed(3)
    W, H = SMALL
    px = W * H
    # the small view comes first: its part of every packed array is the leading one
    mask = torch.zeros(views.P, dtype=torch.uint8, device="cuda")
    target = torch.zeros(3 * views.P, device="cuda")
    mask[:px] = (torch.rand(px, generator=g, device="cuda") < 0.7).to(torch.uint8)
    target[:3 * px] = torch.rand(3 * px, generator=g, device="cuda")
    hits = torch.zeros(N, dtype=torch.int32, device="cuda")
    ma, mw = torch.zeros(N, device="cuda"), torch.zeros(N, device="cuda")
    r.preprocess(p)
    r.bin()
    out = {}
    if kind == "train":
        r.train_step_raster(mask, target, 0.5, 1.0, stats=hits)
        scale = float(views.V)                 # the loss is the mean over the views
    elif kind == "prune":
        r.prune_stats(hits, ma, mw)
    else:
        r.forward(stats=hits, median=True)
        up = lambda n: torch.zeros(n * views.P, device="cuda")
        d = {"dC": up(3), "dA": up(1), "dD": up(1), "dN": up(3), "dS": up(1), "dM": up(1)}
        for k, t in d.items():
            n = (3 if k in ("dC", "dN") else 1) * px
            t[:n] = torch.randn(n, generator=g, device="cuda")
        r.backward_raster(**d)
        out["median"] = r.median_depth[:px].clone()
        scale = 1.0
    if kind != "prune":
        for k, n in (("color", 3), ("alpha", 1), ("depth", 1), ("normal", 3), ("dist", 1), ("n_contrib", 1)):
            out[k] = getattr(r, k)[:n * px].clone()
        out["rec"] = r.grad_rec[:N * 24].clone() * scale
    out["stats"] = (hits, ma, mw)
    return out, views


@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (8, 8), (32, 8)])
@pytest.mark.parametrize("kind", ["train", "eq3"])
def test_records_from_the_scalar_cache_and_from_lds_agree(kind, tile):
    p = _params(11)
    small = _camera((1.0, 0.4, -0.8), SMALL)
    # the large frame looks away from the surfels: no entries, no statistics
    away = _camera((-1.0, 0.2, 0.5), LARGE)
    away.viewmat = away.viewmat.copy()
    away.viewmat[1:] *= -1.0                   # half a turn about x
    alone, _ = _run([small], tile, kind, p)
    beside, views = _run([small, away], tile, kind, p)
    assert views.P > 2_000_000
    for k in alone:
        if k in ("rec", "stats"):
            continue
        assert torch.equal(alone[k], beside[k]), k
    assert torch.equal(alone["stats"][0], beside["stats"][0])
    assert int(alone["stats"][0].sum()) > 0
    a, b = alone["rec"].double(), beside["rec"].double()
    # sums over at most 64 pixels a wave and a few waves a record, in another
    # order: 64 eps of the values' size
    assert float((a - b).norm()) <= 64 * 6e-8 * float(a.norm())
    assert float(a.norm()) > 0.0


@pytest.mark.parametrize("tile", [(16, 16), (8, 8)])
def test_pruning_statistics_agree(tile):
    p = _params(12)
    small = _camera((0.3, 1.0, 0.6), SMALL)
    away = _camera((-1.0, 0.2, 0.5), LARGE)
    away.viewmat = away.viewmat.copy()
    away.viewmat[1:] *= -1.0
    alone, _ = _run([small], tile, "prune", p)
    beside, _ = _run([small, away], tile, "prune", p)
    for a, b in zip(alone["stats"], beside["stats"]):
        assert torch.equal(a, b)
    assert int(alone["stats"][0].sum()) > 0
