"""Row copies of the compaction at the edges of its chunks of 1024 surfels and
of its 16-byte path: widths below, at and beyond four words and the block's
256 threads, and arrays that start off a 16-byte boundary."""
import numpy as np
import pytest
import torch

from paper_2501_08174_amd.raster import compact_surfels

pytestmark = pytest.mark.gpu

WIDTHS = (1, 3, 4, 48, 255, 256, 257, 1028)


@pytest.mark.parametrize("N", [1, 1023, 1024, 1025, 2049, 300_000])
@pytest.mark.parametrize("offset", [0, 1])
def test_rows_match_boolean_indexing(N, offset):
    g = torch.Generator(device="cuda").manual_seed(N + offset)
    widths = WIDTHS if N < 3000 else (1, 4, 5)      # 300,000 surfels: more chunks than one scan round
    arrays = []
    for w in widths:
        flat = torch.rand(N * w + offset, generator=g, device="cuda")
        arrays.append(flat[offset:].view(N, w))
    prune = (torch.rand(N, generator=g, device="cuda") < 0.6).to(torch.uint8)
    out = compact_surfels(prune, arrays)
    keep = prune.cpu().numpy() == 0
    for a, o in zip(arrays, out):
        want = a.cpu().numpy()[keep]
        got = o.cpu().numpy()
        assert got.shape == want.shape
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
