"""The forward where every list is crowded with large primitives, and where most
are short."""
import numpy as np
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer
from tests import gpu_common as GC
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


def test_wide_tiles_of_a_sparse_image():
    """Short lists, 2.7 entries a tile: filtering them for each group cost more
    than it saved (70 us against 54 at 8-pixel tiles)."""
    sc = scenes.room_octahedra(20000, seed=1)
    sc.dists *= 3.0
    cams = [scenes.look_at((8.0, 0.0, 0.0), (0, 0, 0), 3840, 2160)]
    prims = L.Prims.from_scene(sc)
    us = {}
    for tile in (8, 16):
        rast = Rasterizer(sc.kind, sc.n, cams, tile=tile)
        out = rast.forward(prims)
        us[tile] = _best_us(lambda: rast.render(prims, out=out))
    print(f"forward of a sparse 3840x2160 image, {rast.n_pairs} pairs: {us} us", flush=True)
    assert us[16] <= 1.15 * us[8]


@pytest.mark.parametrize("kind", [OCTA, TETRA])
@pytest.mark.parametrize("n,large,opacity", [(1, 1.0, 1.0), (31, 1.0, 0.2), (33, 1.0, 0.05), (64, 0.9, 0.05),
                                             (65, 0.5, 0.1), (200, 1.0, 0.02), (200, 0.97, 0.02), (300, 0.3, 0.05),
                                             (400, 0.0, 1.0)])
def test_exact_rays_together_or_by_rows(kind, n, large, opacity):
    """Exact rays walk a batch as one wave where its rows would gain little:
    all, most, some or none of the primitives cover every quad.  The batches,
    and with them the choice, differ between tile sizes and between a view
    that cuts them off and one that does not; every image is the same bit for
    bit, and the oracle's."""
    import oracle
    print(f"exact rays kind={kind} n={n} large={large} opacity={opacity}", flush=True)
    gen = scenes.uniform_octahedra if kind == OCTA else scenes.uniform_tetrahedra
    sc = gen(n, seed=n + kind, box=0.3, dmin=0.015, dmax=0.03)
    sc.dists[np.random.default_rng(n).permutation(n)[: int(round(large * n))]] *= 20.0
    sc.opacity[:] *= opacity
    cams = [scenes.look_at((0.05, 0.1, -2.0), (0, 0, 0), 45, 37)]
    bg, ref = (0.2, 0.3, 0.1), None
    for tile in (8, 16, 32):
        g = GC.gpu_forward(sc, cams, tile=tile, bg=bg, exact=True, counters=True)
        rast, prims = g["rast"], g["prims"]
        depth = torch.empty(rast.n_pixels, device="cuda")
        plain, with_depth = rast.render(prims, bg), rast.render(prims, bg, depth=depth)
        for a, b, c in zip(plain, with_depth, (g["rgb"], g["T"], g["last"])):
            assert torch.equal(a, b) and np.array_equal(a.cpu().numpy().astype(c.dtype), c)
        O = oracle.OracleScene(sc, cams, tile=tile, exact=True)
        r = O.render(bg=np.asarray(bg))
        r["cams"] = cams
        label = f"together {kind} {n} {large} {tile}"
        GC.compare_images(g, r, label, max_excluded=2e-2)
        GC.compare_last(g, r, label)
        GC.compare_counts(g["counts"], r["counts"], label)
        if ref is None:
            ref = (plain[0], plain[1], depth)
        assert torch.equal(plain[0], ref[0]) and torch.equal(plain[1], ref[1]) and torch.equal(depth, ref[2])
