"""The forward where every list is crowded with large primitives."""
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer
from tests.test_gpu_binning_routes import _best_us

pytestmark = pytest.mark.gpu
OCTA, TETRA = scenes.OCTAHEDRON, scenes.TETRAHEDRON


def _large(kind, n, dmin, dmax, width, height, opacity=1.0):
    gen = scenes.uniform_octahedra if kind == OCTA else scenes.uniform_tetrahedra
    sc = gen(n, seed=n, dmin=dmin, dmax=dmax)
    sc.opacity[:] *= opacity
    return sc, [scenes.look_at((0.3, 0.2, -3.0), (0, 0, 0), width, height)]


@pytest.mark.parametrize("kind", [OCTA, TETRA])
def test_wide_tiles_cost_no_more(kind):
    """16-pixel tiles filter their lists for each 8 x 8 group; what they do
    beyond that has to pay for itself (the outlines' test does for octahedra;
    with it, tetrahedra took 103 us here against 80 at 8-pixel tiles)."""
    sc, cams = _large(kind, 20000, 0.05, 0.3, 1920, 1080)
    prims = L.Prims.from_scene(sc)
    us = {}
    for tile in (8, 16):
        rast = Rasterizer(sc.kind, sc.n, cams, tile=tile)
        out = rast.forward(prims)
        us[tile] = _best_us(lambda: rast.render(prims, out=out))
    print(f"forward of 20000 large primitives, kind {kind}: {us} us", flush=True)
    assert us[16] <= 1.1 * us[8]
