"""Counts read back while something else on the thread or the device is in an
unusual state."""
import ctypes
import threading

import pytest
import torch

from paper_2501_16312_amd import linprim as L
from paper_2501_16312_amd import scenes
from paper_2501_16312_amd.render import Rasterizer

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime this process runs on."""
    torch.cuda.init()
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


MODES = {"global": 0, "thread_local": 1, "relaxed": 2}


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("captured", ["blocking", "nonblocking"])
@pytest.mark.parametrize("on", ["null", "other"])
@pytest.mark.parametrize("thread", ["same", "another"])
def test_while_another_stream_is_captured(mode, captured, on, thread):
    """As a copy and a stream synchronisation: the null stream may be waited
    for; another stream not, where the capture's mode forbids unsafe calls on
    this thread, and then the capture ends in an error too."""
    print(f"read back on the {on} stream, {thread} thread, capture of a {captured} stream, {mode}", flush=True)
    hip = _hip()
    r, want = _binned()
    s, o, g = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1 if captured == "nonblocking" else 0) == 0
    assert hip.hipStreamCreateWithFlags(ctypes.byref(o), 1) == 0
    got = []
    call = lambda: got.append(_pair_count(r, None if on == "null" else o))
    assert hip.hipStreamBeginCapture(s, MODES[mode]) == 0
    if thread == "same":
        call()
    else:
        t = threading.Thread(target=call)
        t.start()
        t.join()
    ended = hip.hipStreamEndCapture(s, ctypes.byref(g))
    hip.hipGetLastError()
    if g.value:
        hip.hipGraphDestroy(g)
    hip.hipStreamDestroy(s)
    refused = on == "other" and (mode == "global" or (mode == "thread_local" and thread == "same"))
    if refused:
        assert got[0][0] == L.ERR_HIP and ended != 0
    else:
        assert got[0] == (L.OK, want) and ended == 0
    assert _pair_count(r, o) == (L.OK, want)
    hip.hipStreamDestroy(o)


@pytest.mark.parametrize("device,pinned,shift", [("cpu", False, 0), ("cpu", False, 4), ("cpu", True, 0),
                                                 ("cpu", True, 4), ("cuda", False, 4)])
def test_status_words_a_kernel_may_not_read(device, pinned, shift):
    """A status block in host memory, or off the 8-byte alignment, is answered
    as the copy answers it: taken, but for host memory that is not pinned."""
    print(f"read back from {device}, pinned {pinned}, {shift} bytes off", flush=True)
    r, want = _binned()
    n, over = ctypes.c_int64(-1), ctypes.c_int32(-1)
    buf = torch.zeros(256 + shift, dtype=torch.uint8, device=device, pin_memory=pinned)
    buf[shift:shift + 64].copy_(r.view_ws[:64])
    torch.cuda.synchronize()
    rc = L.load().linprim_read_status(ctypes.c_void_p(buf.data_ptr() + shift), ctypes.byref(n), ctypes.byref(over),
                                      None)
    _hip().hipGetLastError()           # of a refused copy
    taken = device == "cuda" or pinned
    assert (rc, n.value, over.value) == ((L.OK, want, 0) if taken else (L.ERR_HIP, -1, -1))
    assert _pair_count(r) == (L.OK, want)
