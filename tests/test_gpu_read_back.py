"""Counts read back through pinned slots: several threads, each with its own
stream and population, over many calls; more threads than slots; behind work
longer than the polled wait; and refused under capture, with the stream
usable afterwards."""
import threading

import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer

pytestmark = pytest.mark.gpu


def _rast(n, seed):
    sc = scenes.uniform_octahedra(n, seed=seed, dmin=0.02, dmax=0.08)
    r = Rasterizer(sc.kind, sc.n, [scenes.look_at((0.3, 0.2, -3.0), (0, 0, 0), 320, 200)])
    return r, L.Prims.from_scene(sc)


def _count(r):
    """The pair count, from the status block itself."""
    torch.cuda.synchronize()
    return int(r.view_ws[:8].view(torch.int64).cpu().item())


@pytest.mark.parametrize("threads", [1, 4, 70])
def test_threads_on_their_own_streams(threads):
    print(f"read back: {threads} threads", flush=True)
    made, want = [], []
    for k in range(min(threads, 6)):
        r, prims = _rast(200 + 150 * k, seed=k)
        r.forward(prims)
        made.append((r, prims))
        want.append(_count(r))
    assert len(set(want)) == len(want)
    bad, streams = [], [torch.cuda.Stream() for _ in range(min(threads, 6))]

    def work(t):
        k = t % len(made)
        for _ in range(40):
            with torch.cuda.stream(streams[k]):
                n = L.linprim_pair_count(made[k][0].view_ws)
                m, over = L.linprim_read_status(made[k][0].view_ws)
            if n != want[k] or m != want[k] or over:
                bad.append((t, n, m, over, want[k]))

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not bad, bad[:4]


def test_behind_long_work():
    print("read back behind long work", flush=True)
    r, prims = _rast(500, seed=9)
    r.forward(prims)
    want = _count(r)
    a = torch.zeros(1 << 28, device="cuda")
    for _ in range(20):                 # some 8 ms, well past the polled wait
        a.add_(1.0)
    assert L.linprim_pair_count(r.view_ws) == want
    assert (a[0].item(), a[-1].item()) == (20.0, 20.0)


def test_refused_under_capture():
    print("read back under capture", flush=True)
    r, prims = _rast(300, seed=4)
    r.forward(prims)
    want = _count(r)
    x = torch.zeros(64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1.0)
        with pytest.raises(L.LinPrimError):
            L.linprim_pair_count(r.view_ws)
        with pytest.raises(L.LinPrimError):
            L.linprim_read_status(r.view_ws)
    for k in range(3):
        g.replay()
        assert L.linprim_pair_count(r.view_ws) == want
    torch.cuda.synchronize()
    assert x.eq(3.0).all().item()
