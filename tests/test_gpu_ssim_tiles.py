"""D-SSIM and its gradient at the edges of the 32x32 tiles and of the 11-tap
window, against float64 convolutions."""
import math

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import SsimLoss, ViewBatch

pytestmark = pytest.mark.gpu

W_S = 0.2


def _ssim64(x, y):
    k = torch.arange(-5, 6, dtype=torch.float64, device="cuda")
    g = torch.exp(-k * k / (2.0 * 1.5 * 1.5))
    g = g / g.sum()

    def f(a):
        a = torch.nn.functional.conv2d(a[:, None], g.view(1, 1, 1, 11), padding=(0, 5))
        return torch.nn.functional.conv2d(a, g.view(1, 1, 11, 1), padding=(5, 0))[:, 0]

    mx, my = f(x), f(y)
    vx, vy, cxy = f(x * x) - mx * mx, f(y * y) - my * my, f(x * y) - mx * my
    s = (2 * mx * my + 1e-4) * (2 * cxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
    return s.mean()


@pytest.mark.parametrize("sizes", [[(1, 1)], [(4, 11)], [(31, 33), (33, 31)], [(32, 32)], [(64, 65), (5, 200), (37, 1)],
                                   [(43, 42)] * 9])
def test_edges_of_tiles(sizes):
    cams = [scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -4.0]), W, H) for W, H in sizes]
    views = ViewBatch(cams)
    g = torch.Generator(device="cuda").manual_seed(views.P)
    color = torch.rand(3 * views.P, generator=g, device="cuda").requires_grad_(True)
    target = torch.rand(3 * views.P, generator=g, device="cuda")
    mask = (torch.rand(views.P, generator=g, device="cuda") < 0.8).to(torch.uint8)
    ws = torch.zeros(_lib.workspace_bytes_ssim(views.V, views.host), dtype=torch.uint8, device="cuda")
    total, per = SsimLoss.apply(color, target, mask, views, W_S, ws)
    total.backward()
    c64 = color.detach().double().requires_grad_(True)
    loss, want = 0.0, []
    for v, (W, H) in enumerate(sizes):
        m = mask[views.view_slice(v)].double().view(1, H, W)
        x = m * c64[views.view_slice(v, 3)].view(3, H, W)
        y = m * target.double()[views.view_slice(v, 3)].view(3, H, W)
        s = _ssim64(x, y)
        want.append(float(s.detach()))
        loss = loss + W_S * (1.0 - s) / len(sizes)
    loss.backward()
    # moments of values in [0, 1] carry a few eps; the variances are divided
    # by at least 9e-4: eps / 9e-4 of S per pixel
    tol = 8 * 6e-8 / 9e-4
    assert abs(float(total.detach()) - float(loss.detach())) <= tol
    np.testing.assert_allclose(per[:len(sizes)].cpu().numpy(), want, atol=tol)
    err = (color.grad.double() - c64.grad).norm() / c64.grad.norm()
    assert float(err) <= 10 * tol
    assert math.isfinite(float(err))
