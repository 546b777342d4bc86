"""The forward's walk of a tile's list (records staged in LDS 32 at a time,
each 16-lane row walking the entries that meet its 4 x 4 quad; tiles wider
than a group filter the list 64 entries at a time) at the lengths where a
batch is full, one over or has an odd rest, vs the FP64 oracle on the GPU:
image, transmittance, last blended position, counters and depth map, at the
tolerances of the other forward tests."""
import numpy as np
import pytest
import torch

from paper_2501_16312_amd import scenes
from tests import gpu_common as GC

pytestmark = pytest.mark.gpu
OCTA, TETRA = scenes.OCTAHEDRON, scenes.TETRAHEDRON


@pytest.mark.parametrize("kind,exact", [(OCTA, False), (OCTA, True), (TETRA, False), (TETRA, True)])
@pytest.mark.parametrize("n,tile,faint", [(1, 8, False), (31, 8, True), (32, 16, False), (33, 8, False),
                                          (63, 32, True), (64, 16, True), (65, 16, False), (97, 32, False),
                                          (128, 8, True), (129, 8, True), (160, 8, False), (161, 16, True),
                                          (191, 8, True), (193, 32, True), (400, 16, False)])
def test_quad_walk(kind, exact, n, tile, faint):
    import oracle
    print(f"quad walk kind={kind} exact={exact} n={n} tile={tile} faint={faint}", flush=True)
    gen = scenes.uniform_octahedra if kind == OCTA else scenes.uniform_tetrahedra
    # every primitive lies in the one tile of the image, most of them across
    # only some of its 8 x 8 groups
    d = 3.2 / (0.866 * tile)                       # half-axes of 1.6 to 3.2 pixels
    sc = gen(n, seed=n + tile, box=0.25, dmin=d, dmax=2 * d)
    if faint:
        sc.opacity[:] *= 0.05
    cams = [scenes.look_at((0.05, 0.1, -2.0), (0, 0, 0), tile, tile)]
    bg = (0.2, 0.3, 0.1)
    g = GC.gpu_forward(sc, cams, tile=tile, bg=bg, exact=exact, counters=True)
    assert g["n_pairs"] == n
    O = oracle.OracleScene(sc, cams, tile=tile, exact=exact)
    r = O.render(bg=np.asarray(bg))
    r["cams"] = cams
    label = f"quads {kind} {exact} {n} {tile}"
    GC.compare_images(g, r, label, max_excluded=2e-2)
    GC.compare_last(g, r, label)
    GC.compare_counts(g["counts"], r["counts"], label)
    # without counters, and with the depth map
    rast, prims = g["rast"], g["prims"]
    rgb, T, last = rast.render(prims, bg)
    depth = torch.empty(rast.n_pixels, device="cuda")
    rgb_d, T_d, last_d = rast.render(prims, bg, depth=depth)
    for a, b, c in ((rgb, rgb_d, g["rgb"]), (T, T_d, g["T"]), (last, last_d, g["last"])):
        assert torch.equal(a, b) and np.array_equal(a.cpu().numpy().astype(c.dtype), c)
    d = O.render_depth(bg=np.asarray(bg))
    ok, got = ~d["ill"], depth.cpu().numpy().astype(np.float64)
    assert np.array_equal(got[ok] > 0, d["depth"][ok] > 0)
    assert (np.abs(got - d["depth"]) / np.maximum(d["depth"], 1.0))[ok].max(initial=0.0) <= 1e-5
