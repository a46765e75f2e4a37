"""D-SSIM of a view of more than 2^31 pixels: its last rows give the squared
error and the gradient that the same rows give in a view of 64 rows."""
import ctypes
import math

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import ViewBatch, _ctx, _ptr, _stream

pytestmark = pytest.mark.gpu

W, ROWS = 65535, 24            # the widest view; rows at its end that are not empty


def _ssim(H, x, y):
    """(squared error, gradient of the last ROWS rows times the pixels of the view)."""
    views = ViewBatch([scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -4.0]), W, H)])
    P = views.P
    color, target, grad = (torch.zeros(3 * P, device="cuda") for _ in range(3))
    mask = torch.zeros(P, dtype=torch.uint8, device="cuda")
    last = lambda t: t.view(3, H, W)[:, H - ROWS:]
    last(color).copy_(x)
    last(target).copy_(y)
    mask.view(H, W)[H - ROWS:] = 1
    need = _lib.workspace_bytes_ssim(1, views.host)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = torch.zeros(3, device="cuda")
    _lib.call("sr_ssim_loss", _ctx(color), 1, views.host_ptr, _ptr(views.dev), _ptr(color), _ptr(target), _ptr(mask),
              0.2, _ptr(ws), ctypes.c_size_t(need), _ptr(out), _ptr(grad), _stream())
    se = 10.0 ** (-float(out[1]) / 10.0) * 3.0 * P
    return se, last(grad).double() * P


def test_view_of_more_pixels_than_32_bits_hold():
    H = 32 * 1025
    assert W * (H - ROWS) > 2 ** 31 and W * H < 2 ** 32
    # colours, targets and gradients 12 bytes a pixel, three maps of 12, the mask
    if torch.cuda.mem_get_info()[0] < W * H * (3 * 12 + 3 * 12 + 1) + (8 << 30):
        pytest.skip("needs 170 GB of device memory")
    g = torch.Generator(device="cuda").manual_seed(5)
    x, y = (torch.rand(3, ROWS, W, generator=g, device="cuda") for _ in range(2))
    se, grad = _ssim(64, x, y)
    se_large, grad_large = _ssim(H, x, y)
    torch.cuda.empty_cache()
    want = float(((x - y).double() ** 2).sum())
    # 39 decibels in float32, a few units of the last place (3.8e-6) off, and 10^(decibels / 10) of them
    tol = 10 * 3.8e-6 * math.log(10.0) / 10.0
    assert abs(se - want) <= tol * want and abs(se_large - want) <= tol * want
    # the same tiles and windows but for the factor 1 / pixels: some 30 roundings
    # of terms that cancel to no less than a hundredth of their size
    assert float(grad.abs().max()) > 0.0
    assert float((grad_large - grad).abs().max()) <= 100 * 30 * 6e-8 * float(grad.abs().max())
