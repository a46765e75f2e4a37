"""Launches of one D-SSIM call, counted in a captured graph: a single view's
totals need no launch of their own."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2501_08174_amd import _lib, scenes
from paper_2501_08174_amd.raster import ViewBatch, _ctx, _ptr, _stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,with_grad,most", [(1, True, 3), (1, False, 2), (3, True, 4)])
def test_kernels_of_a_call(V, with_grad, most):
    views = ViewBatch([scenes.make_camera(np.eye(3), np.array([0.0, 0.0, -4.0]), 50, 40 + v) for v in range(V)])
    g = torch.Generator(device="cuda").manual_seed(1)
    color, target = (torch.rand(3 * views.P, generator=g, device="cuda") for _ in range(2))
    mask = torch.ones(views.P, dtype=torch.uint8, device="cuda")
    need = _lib.workspace_bytes_ssim(V, views.host)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")

    def call():
        out, grad = torch.zeros(2 * V + 1, device="cuda"), torch.zeros(3 * views.P, device="cuda")
        torch.cuda.synchronize()
        return out, grad

    def run(out, grad):
        _lib.call("sr_ssim_loss", _ctx(color), V, views.host_ptr, _ptr(views.dev), _ptr(color), _ptr(target),
                  _ptr(mask), 0.2, _ptr(ws), ctypes.c_size_t(need), _ptr(out), _ptr(grad) if with_grad else None,
                  _stream())

    eager = call()
    run(*eager)
    torch.cuda.synchronize()
    captured = call()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        run(*captured)
    n = ctypes.c_size_t()
    # the HIP runtime that the library is linked to
    assert _lib.lib().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert 0 < n.value <= most
    graph.instantiate()
    for _ in range(2):                         # the gradient is added to: clear it between the replays
        captured[1].zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured[0], eager[0]) and torch.equal(captured[1], eager[1])
