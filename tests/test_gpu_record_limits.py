"""The launches' sizes at which the compositing kernels turn from records in LDS
to records through the scalar cache (waves per SIMD of the device): one tile
below the limit and at it, a view gives the same images, decisions and record
gradients."""
import pytest
import torch

from tests.test_gpu_records import SMALL, _camera, _params, _run

pytestmark = pytest.mark.gpu

LIMITS = {"eq3": 10, "colour": 14, "train": 18, "prune": 28}


def _away(tiles, tile):
    """A strip of so many tiles that looks away from the surfels."""
    c = _camera((-1.0, 0.2, 0.5), (tile[0] * tiles, tile[1]))
    c.viewmat = c.viewmat.copy()
    c.viewmat[1:] *= -1.0
    return c


@pytest.mark.parametrize("tile", [(16, 16), (32, 8)])
@pytest.mark.parametrize("kind", list(LIMITS))
def test_one_tile_below_and_at_the_limit(kind, tile, monkeypatch):
    simds = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    tiles = LIMITS[kind] * simds * 64 // (tile[0] * tile[1])
    if kind == "colour":
        from paper_2501_08174_amd.raster import Rasterizer
        full = Rasterizer.backward_raster
        monkeypatch.setattr(Rasterizer, "backward_raster",
                            lambda r, dC, dA, **rest: full(r, dC=dC, dA=dA))
    p = _params(21)
    small = _camera((1.0, 0.4, -0.8), SMALL)
    rest = tiles - -(-SMALL[0] // tile[0]) * -(-SMALL[1] // tile[1])
    got = []
    for n in (rest - 1, rest):
        strips = [n - n // 4 * 3] + [n // 4] * 3          # widths below 65536 pixels
        out, views = _run([small] + [_away(k, tile) for k in strips], tile, "eq3" if kind == "colour" else kind, p)
        assert views.T == tiles - (n < rest)
        got.append(out)
    below, at = got
    for k in below:
        if k not in ("rec", "stats"):
            assert torch.equal(below[k], at[k]), k
    for a, b in zip(below["stats"], at["stats"]):
        assert torch.equal(a, b)
    assert int(at["stats"][0].sum()) > 0
    if kind != "prune":
        a, b = below["rec"].double(), at["rec"].double()
        # the same terms, summed over a record's waves and tiles in another order
        assert float((a - b).norm()) <= 64 * 6e-8 * float(a.norm())
        assert float(a.norm()) > 0.0
