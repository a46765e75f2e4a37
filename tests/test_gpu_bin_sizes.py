"""The binning at the sizes where its passes change their blocks: one block up
to 1024, 4096 and 8192 pairs, then 1024 pairs a block, 256 Ki and 2 Mi pairs a radix grid, 16 Mi instances of capacity an
emission block.  The sorted instances are checked against what defines them:
strictly increasing (group, depth, surfel), every surfel once per group its
rectangle meets, the depth its own, and the ranges the runs of the groups."""
import math

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import scenes
from paper_2501_08174_amd.raster import Params, Rasterizer, ViewBatch

pytestmark = pytest.mark.gpu


def _rasterizer(N, size, scale):
    g = torch.Generator(device="cuda").manual_seed(N)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")
    c = np.array([0.5, -0.3, -3.0])
    views = ViewBatch([scenes.make_camera(scenes.look_at_rotation(c), c, *size)])
    p = Params(r(N, 3) * 4.0 - 2.0, torch.exp(math.log(scale) + r(N, 2)), torch.randn(N, 4, generator=g, device="cuda"),
               r(N), torch.zeros(N, 1, 3, device="cuda"))
    rast = Rasterizer(N, views, 0)
    return rast, p, views


@pytest.mark.parametrize("N,size,scale,capacity", [
    (1, (64, 64), 0.1, None), (1023, (200, 120), 0.02, None), (1024, (200, 120), 0.02, None),
    (1025, (200, 120), 0.02, None), (4096, (300, 200), 0.02, None), (4097, (300, 200), 0.02, None),
    (8192, (300, 200), 0.01, None), (8193, (300, 200), 0.01, None),
    ((1 << 18) - 1, (300, 200), 0.002, None), (1 << 18, (300, 200), 0.002, None),
    ((1 << 18) + 1, (300, 200), 0.002, None), ((1 << 21) + 1, (260, 130), 0.001, None),
    (5000, (640, 480), 0.05, (16 << 20) - 5), (5000, (640, 480), 0.05, (16 << 20) + 1)])
def test_sorted_instances(N, size, scale, capacity):
    rast, p, views = _rasterizer(N, size, scale)
    need = rast.plan_capacity(p)
    if capacity is not None:
        rast.set_capacity(capacity)
    keys = torch.zeros(max(rast.capacity, 1), dtype=torch.int64, device="cuda")
    rast.bin(keys64=keys)
    vis, got, stored, status = rast.status()
    assert got == need == stored and status == 0
    keys, vals = keys[:stored], rast.vals[:stored].long() & 0xFFFFFF
    group, depth = keys >> 32, keys & 0xFFFFFFFF
    assert torch.equal(depth, rast.depth_key.long()[vals] & 0xFFFFFFFF)
    later = (keys[1:] > keys[:-1]) | ((keys[1:] == keys[:-1]) & (vals[1:] > vals[:-1]))
    assert bool(later.all())
    # groups of 64 x 64 pixels met by every visible rectangle (x_lo, x_hi, y_lo, y_hi)
    rc = (rast.rect.view(N, 4).long() & 0xFFFF) >> 6
    seen = rast.tiles_touched != 0
    met = (rc[:, 1] - rc[:, 0] + 1) * (rc[:, 3] - rc[:, 2] + 1) * seen
    assert int(seen.sum()) == vis and int(met.sum()) == need
    assert torch.equal(torch.bincount(vals, minlength=N), met)
    gx = group % views.host[0].groups_x
    gy = group // views.host[0].groups_x
    r = rc[vals]
    assert bool(((gx >= r[:, 0]) & (gx <= r[:, 1]) & (gy >= r[:, 2]) & (gy <= r[:, 3])).all())
    # ranges: the run of the tile's group, [0, 0) for an empty one
    cam = views.host[0]
    tiles = torch.arange(views.T, device="cuda")
    tg = (tiles // cam.tiles_x // 4) * cam.groups_x + tiles % cam.tiles_x // 4
    lo, hi = torch.searchsorted(group, tg), torch.searchsorted(group, tg, right=True)
    want = torch.where((lo < hi)[:, None], torch.stack([lo, hi], 1), torch.zeros(1, 2, dtype=lo.dtype, device="cuda"))
    assert torch.equal(rast.ranges[:2 * views.T].view(-1, 2).long(), want)


@pytest.mark.parametrize("T", [1, 1023, 1024, 1025, 4096, 4097, 8192, 8193])
def test_tile_order(T):
    """Tiles by descending cost class (16 per octave above 16), ties by id."""
    import ctypes

    from paper_2501_08174_amd import _lib
    from paper_2501_08174_amd._lib import call

    g = torch.Generator(device="cuda").manual_seed(T)
    cost = torch.exp(torch.rand(T, generator=g, device="cuda", dtype=torch.float64) * 20.0).long()
    cost[torch.rand(T, generator=g, device="cuda") < 0.3] = 0
    c32 = cost.to(torch.int32)
    n = ctypes.c_size_t(0)
    call("sr_tile_order_workspace_size", T, ctypes.byref(n))
    ws = torch.zeros(max(n.value, 1), dtype=torch.uint8, device="cuda")
    order = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    ctx = _lib.default_context(0)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    call("sr_tile_order", ctx.ptr, T, ptr(c32), ptr(ws), ws.numel(), ptr(order),
         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    c = cost.cpu().numpy()
    e = np.floor(np.log2(np.maximum(c, 1))).astype(np.int64)
    cls = np.where(c < 16, c, (e - 3) * 16 + ((c >> np.maximum(e - 4, 0)) & 15))
    want = np.lexsort((np.arange(T), -cls))
    assert np.array_equal(order.cpu().numpy(), want)
