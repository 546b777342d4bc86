"""Both routes of the default sort (tile counters, and emission with tile-bit
radix passes for larger pair capacities) on the same scenes, vs the FP64
oracle bit for bit: few primitives of many tiles, runs over the whole image,
lists of every length, tiles of 8, 16 and 32, several views, nothing visible."""
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer
from tests.test_gpu_tile_counters import _check

pytestmark = pytest.mark.gpu
ROUTES = {"counters": 131072, "radix": 131073}     # pair capacity


def _made(kind, n, dmin, dmax, width, height, views, behind=False):
    gen = scenes.uniform_octahedra if kind == 0 else scenes.uniform_tetrahedra
    sc = gen(n, seed=n, dmin=dmin, dmax=dmax)
    at = (0, 0, -9.0) if behind else (0, 0, 0)
    cams = [scenes.look_at((0.1 + 0.05 * v, 0.2, -3.0), at, width, height) for v in range(views)]
    return sc, cams


SCENES = [
    # n, distances, image, tile, views
    (1, 1.0, 1.1, 333, 322, 8, 1),         # one run of more than 1024 tiles
    (3, 0.9, 1.4, 501, 399, 8, 1),
    (40, 0.4, 1.2, 333, 322, 8, 1),        # huge runs beside long ones
    (300, 0.2, 0.6, 400, 300, 8, 1),
    (700, 0.2, 0.5, 400, 300, 16, 1),
    (60, 0.5, 1.5, 161, 119, 8, 16),
    (900, 0.02, 0.5, 203, 150, 16, 3),
    (9000, 0.02, 0.3, 65, 63, 32, 1),      # lists beyond the LDS sort
    (2500, 0.02, 0.3, 131, 97, 32, 2),
    (130, 0.3, 0.9, 701, 64, 8, 1),
]


@pytest.mark.parametrize("route", list(ROUTES))
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n,dmin,dmax,width,height,tile,views", SCENES)
def test_routes(route, kind, n, dmin, dmax, width, height, tile, views):
    import oracle
    print(f"binning by {route}: kind={kind} n={n} {width}x{height} tile={tile} views={views}", flush=True)
    sc, cams = _made(kind, n, dmin, dmax, width, height, views)
    s = oracle.OracleScene(sc, cams, tile=tile).sort()
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=tile, headroom=1.0)
    rast.reserve_pairs(ROUTES[route])
    rast.preprocess(prims)
    assert rast.max_pairs == ROUTES[route]
    for _ in range(2):
        rast.bin_sort(prims)
        _check(rast, prims, s)


@pytest.mark.parametrize("route", list(ROUTES))
def test_nothing_visible(route):
    print(f"binning by {route}: nothing visible", flush=True)
    sc, cams = _made(0, 2000, 0.01, 0.02, 320, 200, 2, behind=True)
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=8, headroom=1.0)
    rast.reserve_pairs(ROUTES[route])
    rast.preprocess(prims)
    rast.bin_sort(prims)
    assert rast.n_pairs == 0
    assert rast.debug_arrays(prims)["ranges"].eq(0).all()


def _best_us(f, calls=20, tries=5):
    f()
    best = float("inf")
    for _ in range(tries):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / calls * 1e3)
    return best


@pytest.mark.parametrize("n,dmin,dmax", [(40, 0.4, 1.2), (700, 0.2, 0.6)])
def test_counters_are_chosen_where_they_are_faster(n, dmin, dmax):
    """Few primitives of many tiles are where the counters' work splits worst
    over the chip (with 64 slots to a wave: 108 and 149 us against 68)."""
    sc, cams = _made(0, n, dmin, dmax, 640, 480, 1)
    prims = L.Prims.from_scene(sc)
    us = {}
    for route, capacity in ROUTES.items():
        rast = Rasterizer(sc.kind, sc.n, cams, tile=8, headroom=1.0)
        rast.reserve_pairs(capacity)
        rast.preprocess(prims)
        us[route] = _best_us(lambda: rast.bin_sort(prims))
    print(f"bin_sort of {n} octahedra, {rast.n_pairs} pairs: {us}", flush=True)
    assert us["counters"] <= us["radix"]
