"""Binning by tile counters and the scan that reads the slots before a block
itself: sorted pairs, ranges and both render orders at the tile counts, slot
counts and view counts where they begin, end and hand over to the radix
passes, vs the FP64 oracle and the orders' definitions, bit for bit; and the
state they leave for another bin_sort on the same preprocessing."""
import numpy as np
import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer
from tests import gpu_common as GC

pytestmark = pytest.mark.gpu
# classes of list length of the backward order; parts of the forward's
BOUNDS = np.array([192, 128, 96, 72, 56, 48, 40, 32, 26, 20, 16, 12, 8, 4, 0])
PARTS = np.array([128, 72])


def _orders(rast, prims, n_tiles):
    ptr = L.linprim_debug_pointers(prims, rast.cams_c, rast.tune, rast.view_ws, rast.pair_ws, rast.max_pairs)
    base = rast.view_ws.data_ptr()
    take = lambda k: rast.view_ws[ptr[k] - base: ptr[k] - base + 4 * n_tiles].view(torch.int32).cpu().numpy()
    return take("order_fwd"), take("order_bwd")


def _check(rast, prims, s):
    dbg = rast.debug_arrays(prims)
    assert rast.n_pairs == len(s["keys"])
    assert np.array_equal(dbg["keys"].numpy().view(np.uint64), s["keys"])
    assert np.array_equal(dbg["values"].numpy().view(np.uint32), s["values"])
    rg = dbg["ranges"].numpy().view(np.uint32).astype(np.int64)
    length = s["ranges"][:, 1] - s["ranges"][:, 0]
    assert np.array_equal(rg[length > 0], s["ranges"][length > 0])
    assert np.all(rg[length == 0] == 0)
    fwd, bwd = _orders(rast, prims, len(rg))
    cls = (length[:, None] <= BOUNDS).sum(1)
    part = (length[:, None] <= PARTS).sum(1)
    assert np.array_equal(bwd, np.argsort(cls, kind="stable"))
    assert np.array_equal(fwd, np.argsort(part, kind="stable"))


def _scene(kind, n, seed):
    gen = scenes.uniform_octahedra if kind == 0 else scenes.uniform_tetrahedra
    sc = gen(n, seed=seed, dmin=0.02, dmax=0.08)
    sc.dists[: max(1, n // 500)] *= 8.0          # a few cover many tiles (a whole wave writes them)
    return sc


# (tiles across, tiles down, tile, views): 1 tile, around 1024, 8192 and just beyond
@pytest.mark.parametrize("tx,ty,tile,views", [(1, 1, 8, 1), (31, 33, 8, 1), (32, 32, 8, 1), (25, 41, 8, 1),
                                              (64, 64, 8, 2), (64, 43, 8, 3), (40, 30, 16, 1), (20, 17, 32, 2)])
@pytest.mark.parametrize("kind", [0, 1])
def test_tile_counts(kind, tx, ty, tile, views):
    import oracle
    print(f"tile counters kind={kind} {tx}x{ty} tiles of {tile}, {views} views", flush=True)
    sc = _scene(kind, 1500, seed=tx + ty)
    cams = [scenes.look_at((0.3 * v, 0.2, -3.0 + 0.2 * v), (0, 0, 0), tx * tile - 3, ty * tile - 2)
            for v in range(views)]
    s = oracle.OracleScene(sc, cams, tile=tile).sort()
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=tile)
    rast.preprocess(prims)
    rast.bin_sort(prims)
    _check(rast, prims, s)
    # again on the same preprocessing
    rast.bin_sort(prims)
    _check(rast, prims, s)


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 32768, 32769])
def test_slot_counts(n):
    import oracle
    print(f"slots {n}", flush=True)
    sc = _scene(0, n, seed=n)
    cams = [scenes.look_at((0.1, 0.2, -3.0), (0, 0, 0), 97, 71)]
    O = oracle.OracleScene(sc, cams, tile=8)
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=8)
    rast.preprocess(prims)
    rast.bin_sort(prims)
    dbg = rast.debug_arrays(prims)
    tiles = O.prep(0)["tiles"].astype(np.int64)
    assert np.array_equal(dbg["tiles"].numpy(), tiles)
    assert np.array_equal(dbg["offsets"].numpy(), np.cumsum(tiles) - tiles)
    _check(rast, prims, O.sort())


def test_overflow_then_larger():
    import oracle
    print("overflow, then a larger capacity, then the radix passes", flush=True)
    sc = _scene(0, 3000, seed=3)
    cams = [scenes.look_at((0.1, 0.2, -3.0), (0, 0, 0), 150, 130)]
    s = oracle.OracleScene(sc, cams, tile=8).sort()
    prims = L.Prims.from_scene(sc)
    rast = Rasterizer(sc.kind, sc.n, cams, tile=8)
    rast.reserve_pairs(100)
    rast.preprocess(prims, sync_count=False)
    rast.bin_sort(prims)
    needed, overflow = rast.status()
    assert overflow and needed == len(s["keys"])
    rast.reserve_pairs(needed)
    rast.n_pairs = needed
    rast.bin_sort(prims)
    _check(rast, prims, s)
    # a capacity beyond the counters' range takes the radix passes, and back
    big = Rasterizer(sc.kind, sc.n, cams, tile=8)
    big.reserve_pairs(300_000)
    big.preprocess(prims)
    big.bin_sort(prims)
    _check(big, prims, s)
    big.max_pairs = 0
    big.reserve_pairs(needed)
    big.bin_sort(prims)
    _check(big, prims, s)
