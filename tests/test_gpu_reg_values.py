"""The 2DGS regularisers' gradients for values at the ends of the range:
quotients by alphas whose reciprocal overflows, and depths that are not
numbers."""
import numpy as np
import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import RegularizerLoss, ViewBatch

pytestmark = pytest.mark.gpu

W, H = 64, 48
W_NORMAL = 0.05


def _grads(alpha, depth, normal, median=None):
    views = ViewBatch([scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -4.0]), W, H)])
    maps = [alpha, depth, normal, torch.zeros(W * H, device="cuda")] + ([] if median is None else [median])
    maps = [m.clone().requires_grad_(True) for m in maps]
    ws = torch.zeros(_lib.workspace_bytes_loss(1, views.host), dtype=torch.uint8, device="cuda")
    total, _ = RegularizerLoss.apply(*maps[:4], views, 0.0, W_NORMAL, ws, *maps[4:])
    total.backward()
    return [m.grad.cpu().numpy() for m in maps]


def _maps(seed):
    rng = np.random.default_rng(seed)
    z = (3.0 + 0.5 * rng.random(W * H)).astype(np.float32)
    normal = torch.tensor((rng.random(3 * W * H) - 0.5).astype(np.float32), device="cuda")
    return rng, z, normal


# the smallest subnormal, subnormals whose reciprocal overflows and whose it
# does not, normal numbers, and numbers whose reciprocal is subnormal
RANGES = [(1.4e-45, 1e-44), (1e-44, 2.9e-39), (2.9e-39, 1.2e-38), (1.2e-38, 1e-30), (1e-30, 1.0), (1.0, 1e37)]


@pytest.mark.parametrize("lo,hi", RANGES)
def test_quotients_by_alpha(lo, hi):
    """dL/dD = s / A and dL/dA = g - (s D / A) / A are the rounded quotients of
    s, the gradient by the point's depth (that of the median map)."""
    rng, z, normal = _maps(1)
    a = np.exp(rng.uniform(np.log(lo), np.log(hi), W * H)).astype(np.float32)
    d = (z * a).astype(np.float32)
    assert (a > 0).all()
    alpha, depth = torch.tensor(a, device="cuda"), torch.tensor(d, device="cuda")
    with np.errstate(all="ignore"):
        point = d / a
    assert np.isfinite(point).all()
    gA0, _, _, _, s = _grads(alpha, depth, normal, torch.tensor(point, device="cuda"))
    gA, gD, _, _ = _grads(alpha, depth, normal)
    assert np.isfinite(s).all() and (s != 0).any()
    with np.errstate(all="ignore"):
        np.testing.assert_array_equal(gD, s / a)
        np.testing.assert_array_equal(gA, gA0 - (s * point) / a)


@pytest.mark.parametrize("a", [1.4e-45, 1e-39, 2.9e-39, 1e-20])
def test_zero_gradient_of_any_alpha(a):
    """Without a normal there is no gradient by the depth, whatever the alpha."""
    _, z, normal = _maps(2)
    alpha = torch.full((W * H,), a, device="cuda")
    gA, gD, _, _ = _grads(alpha, alpha * torch.tensor(z, device="cuda"), torch.zeros_like(normal))
    assert not gD.any()
    np.testing.assert_array_equal(gA, np.float32(W_NORMAL) * (np.float32(1) / np.float32(W * H)))


@pytest.mark.parametrize("of", ["depth", "median"])
def test_depth_that_is_no_number(of):
    """A NaN depth makes the two tangent vectors that it takes part in NaN, and
    with them the points of the other tangent of those normals: the four
    diagonal neighbours.  The points two pixels away are passed vectors of the
    finite tangent alone."""
    _, z, normal = _maps(3)
    x, y = 30, 20
    one, bad = torch.ones(W * H, device="cuda"), torch.tensor(z, device="cuda")
    bad[y * W + x] = float("nan")
    grads = _grads(one, bad, normal) if of == "depth" else _grads(one, one, normal, bad)
    got = ~np.isfinite(grads[1 if of == "depth" else 4].reshape(H, W))
    want = np.zeros_like(got)
    want[[y - 1, y - 1, y + 1, y + 1], [x - 1, x + 1, x - 1, x + 1]] = True
    np.testing.assert_array_equal(got, want)
