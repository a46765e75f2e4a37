"""Record gradients of splats that reach a single pixel: the sums weighted
with the pixel's position are then one product each, so their ratio to the
plain sum is the pixel's offset from the projected centre, whatever the errors
of the factors.  All pixels of the tiles take part, the corners included."""
import numpy as np
import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import Params, Rasterizer, ViewBatch

pytestmark = pytest.mark.gpu

W, H, F, Z = 64, 32, 60.0, 4.0
LARGE = (1640, 1290)


def _camera(size, away=False):
    c = scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -Z]), *size)
    c.fx = c.fy = F
    c.cx, c.cy = size[0] / 2.0, size[1] / 2.0
    if away:                                   # half a turn about x: the splats are behind it
        c.viewmat = c.viewmat.copy()
        c.viewmat[1:] *= -1.0
    return c


def _splats(scale_px, seed):
    """One splat a pixel, facing the camera, its centre within 0.15 of the
    pixel's, of an opacity that passes the cutoff up to 0.3 of its scale (in
    the plane) or 0.22 pixels (the low-pass)."""
    rng = np.random.default_rng(seed)
    i, j = np.meshgrid(np.arange(W), np.arange(H))
    px = np.stack([i, j], -1).reshape(-1, 2) + 0.5 + rng.uniform(-0.15, 0.15, (W * H, 2))
    n = W * H
    t = lambda a: torch.tensor(np.asarray(a, np.float32), device="cuda")
    means = np.concatenate([(px - [W / 2, H / 2]) * Z / F, np.zeros((n, 1))], 1)
    quats = np.tile([1.0, 0.0, 0.0, 0.0], (n, 1))
    return Params(t(means), t(np.full((n, 2), scale_px * Z / F)), t(quats), t(np.full(n, 1.05 / 255.0)),
                  t(0.3 * rng.standard_normal((n, 1, 3))))


@pytest.mark.parametrize("beside", [False, True])             # records from LDS, through the scalar cache
@pytest.mark.parametrize("kind", ["train", "colour", "depth"])
@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (8, 8), (32, 8)])
@pytest.mark.parametrize("scale", [0.9, 0.2])                 # in the plane, the low-pass
def test_position_sums_of_one_pixel(scale, tile, kind, beside):
    p = _splats(scale, 7)
    n = W * H
    views = ViewBatch([_camera((W, H))] + ([_camera(LARGE, away=True)] if beside else []), tile=tile)
    r = Rasterizer(n, views, 0)
    r.plan_capacity(p)
    r.preprocess(p)
    r.bin()
    g = torch.Generator(device="cuda").manual_seed(2)
    up = lambda k: torch.randn(k * views.P, generator=g, device="cuda")
    if kind == "train":
        mask = torch.ones(views.P, dtype=torch.uint8, device="cuda")
        r.train_step_raster(mask, up(3), 0.5, 1.0)
    else:
        r.forward()
        more = dict(dD=up(1), dN=up(3), dS=up(1)) if kind == "depth" else {}
        r.backward_raster(dC=up(3), dA=up(1), **more)
    rec = r.grad_rec[:n * _lib.SR_GRAD_STRIDE].view(n, _lib.SR_GRAD_STRIDE).double().cpu().numpy()
    geom = r.geom[:n * _lib.SR_GEOM_STRIDE].view(n, _lib.SR_GEOM_STRIDE).double().cpu().numpy()
    hit = r.n_contrib[:n].cpu().numpy() > 0
    assert hit.all() and (rec[:, 11] != 0).mean() > 0.99
    i, j = np.meshgrid(np.arange(W), np.arange(H))
    dx, dy = i.reshape(-1) + 0.5 - geom[:, 9], j.reshape(-1) + 0.5 - geom[:, 10]
    assert np.abs(dx).max() < 0.2 and np.abs(dy).max() < 0.2
    eps = 2.0 ** -23          # a rounded product, and the rounding of the offset
    worst = lambda a, b: float((np.abs(a - b) / np.maximum(np.abs(b), 1e-30)).max())
    if scale > 0.5:
        for k in range(3):    # dA, dB against dC'
            assert (rec[:, 6 + k] != 0).any()
            assert worst(rec[:, k], rec[:, 6 + k] * dx) <= eps
            assert worst(rec[:, 3 + k], rec[:, 6 + k] * dy) <= eps
    else:
        assert (rec[:, 9] != 0).any()
        assert worst(rec[:, 10] * dx, rec[:, 9] * dy) <= 2 * eps
