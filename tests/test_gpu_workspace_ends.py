"""Tile order and binning at the sizes where their block sizes change, in
workspaces of exactly the size asked for: the results hold and nothing is
written behind the end."""
import ctypes

import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import Params, Rasterizer, ViewBatch, _ctx, _ptr, _stream

pytestmark = pytest.mark.gpu

GUARD = 1 << 16


def _guarded(n):
    return torch.full((n + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("T", [8193, 65788, 1 << 18, (1 << 18) + 1, 1 << 21, (1 << 21) + 1])
def test_tile_order(T):
    g = torch.Generator(device="cuda").manual_seed(T)
    cost = torch.randint(0, 16, (T,), generator=g, device="cuda", dtype=torch.int32)      # exact classes
    order = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    n = ctypes.c_size_t()
    _lib.call("sr_tile_order_workspace_size", T, ctypes.byref(n))
    ws = _guarded(n.value)
    _lib.call("sr_tile_order", _ctx(cost), T, _ptr(cost), _ptr(ws), n, _ptr(order), _stream())
    assert torch.equal(order.long(), torch.sort(cost, descending=True, stable=True).indices)
    assert bool((ws[n.value:] == 0xA5).all())


@pytest.mark.parametrize("capacity", [1 << 18, (1 << 18) + 1, 1 << 21, (1 << 21) + 1, 1 << 24, (1 << 24) + 1])
def test_binning(capacity):
    sc = scenes.make_random_scene(3, 20000, n_views=2, width=[200, 130], height=[150, 97], sh_degree=0,
                                  scale_range=(0.005, 0.3))
    views = ViewBatch(sc.cams)
    r = Rasterizer(sc.n, views, 0, sh_stride=sc.sh.shape[1])
    need = r.plan_capacity(Params.from_scene(sc))
    assert need < 1 << 18
    r.bin()
    want, ranges = r.vals[:need].clone(), r.ranges.clone()
    size = _lib.workspace_bytes_bin(sc.n, views.V, capacity)
    r.ws, r.ws_bytes, r.capacity = _guarded(size), size, capacity
    r.vals = torch.full((capacity,), -1, dtype=torch.int32, device="cuda")
    r.ranges.fill_(-1)
    r.bin()
    assert r.check_capacity() == need
    assert torch.equal(r.vals[:need], want) and torch.equal(r.ranges, ranges)
    assert bool((r.ws[size:] == 0xA5).all())
