"""Counts read back while something else on the thread or the device is in an
unusual state."""
import ctypes

import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime this process runs on."""
    torch.zeros(1, device="cuda")
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return ctypes.CDLL(path)


def _binned():
    sc = scenes.uniform_octahedra(300, seed=1, dmin=0.02, dmax=0.08)
    r = Rasterizer(sc.kind, sc.n, [scenes.look_at((0.3, 0.2, -3.0), (0, 0, 0), 320, 200)])
    r.forward(L.Prims.from_scene(sc))
    torch.cuda.synchronize()
    return r, int(r.view_ws[:8].view(torch.int64).cpu().item())


def _pair_count(r, stream=None):
    """Status and count as the C entry point gives them."""
    n = ctypes.c_int64(-1)
    rc = L.load().linprim_pair_count(ctypes.c_void_p(r.view_ws.data_ptr()), ctypes.byref(n), stream)
    return rc, n.value


def test_error_pending_from_another_call():
    """An error that an earlier, unrelated call left on the thread is neither
    taken for the read-back's own nor taken away from whoever asks for it."""
    print("read back with a pending error", flush=True)
    hip = _hip()
    r, want = _binned()
    hip.hipGetLastError()
    bad = hip.hipSetDevice(9999)
    assert bad != 0
    try:
        assert _pair_count(r) == (L.OK, want)
        assert hip.hipPeekAtLastError() == bad
    finally:
        hip.hipGetLastError()
    assert _pair_count(r) == (L.OK, want)
