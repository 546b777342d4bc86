"""The forward's outline test (tiles wider than a group, batches whose quads
have many entries): images, transmittance, last blended positions and depth
maps equal those of the counted render, which evaluates every rectangle, and
those of 8-pixel tiles (neither takes the test), bit for bit, for needles,
plates and compact primitives at batch sizes on both sides of its threshold;
and the depth map is the oracle's."""
import numpy as np
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer

pytestmark = pytest.mark.gpu
OCTA, TETRA = scenes.OCTAHEDRON, scenes.TETRAHEDRON


def _scene(kind, n, shape, seed):
    gen = scenes.uniform_octahedra if kind == OCTA else scenes.uniform_tetrahedra
    sc = gen(n, seed=seed, box=0.5, dmin=0.02, dmax=0.05)
    sc.opacity[:] *= 0.2
    if shape == "needle":
        sc.dists[:, 0] *= 12.0
    elif shape == "plate":
        sc.dists[:, 1:] *= 8.0
        sc.dists[:, 0] *= 0.2
    return sc


def _render(sc, cams, tile, count=False):
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=tile)
    bg = (0.2, 0.3, 0.1)
    cnt = torch.zeros(3, dtype=torch.int64, device="cuda") if count else None
    rgb, T, last = rast.forward(prims, bg, counters=cnt)
    depth = torch.empty(rast.n_pixels, device="cuda")
    if not count:
        rgb_d, T_d, last_d = rast.render(prims, bg, depth=depth)
        assert torch.equal(rgb, rgb_d) and torch.equal(T, T_d) and torch.equal(last, last_d)
    return rgb, T, last, depth


@pytest.mark.parametrize("shape", ["needle", "plate", "compact"])
@pytest.mark.parametrize("kind", [OCTA, TETRA])
@pytest.mark.parametrize("n", [19, 33, 200, 1500])
def test_outline(kind, shape, n):
    import oracle
    print(f"outline kind={kind} shape={shape} n={n}", flush=True)
    sc = _scene(kind, n, shape, seed=n)
    cams = [scenes.look_at((0.05, 0.1, -2.0), (0, 0, 0), 45, 37)]
    ref = _render(sc, cams, 8)
    for tile in (16, 32):
        got = _render(sc, cams, tile)
        counted = _render(sc, cams, tile, count=True)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]) and torch.equal(got[3], ref[3])
        for a, b in zip(got[:3], counted[:3]):
            assert torch.equal(a, b)
        d = oracle.OracleScene(sc, cams, tile=tile).render_depth(bg=np.asarray((0.2, 0.3, 0.1)))
        ok, dep = ~d["ill"], got[3].cpu().numpy().astype(np.float64)
        assert np.array_equal(dep[ok] > 0, d["depth"][ok] > 0)
        assert (np.abs(dep - d["depth"]) / np.maximum(d["depth"], 1.0))[ok].max(initial=0.0) <= 1e-5
