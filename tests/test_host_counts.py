"""Host side of the entry points that read counts back, on the CPU, against a
stand-in for the HIP runtime (fake_hip.cpp), each in a process of its own."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2501_16312_amd import build
from paper_2501_16312_amd import linprim as L

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, sys
fake = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL({lib!r})
get = lambda name: ctypes.c_int.in_dll(fake, name).value
OK = 0
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    if not os.path.exists(build.LIB):
        build.build()
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run([cxx, "-O1", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)

    def go(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE.format(fake=so, lib=build.LIB) + body], capture_output=True,
                           text=True, timeout=60)
        assert r.returncode == 0, r.stdout + r.stderr

    return go


def test_densify_noalloc_allocates_nothing(run):
    """... as the first call of a process, and after a call that polls."""
    run("""
class State(ctypes.Structure):
    _fields_ = [(f, ctypes.c_void_p) for f in ("means", "quats", "dists", "opacity", "sh")] + \\
               [("exp_avg", ctypes.c_void_p * 5), ("exp_avg_sq", ctypes.c_void_p * 5)]
buf = (ctypes.c_float * 4096)()
at = ctypes.addressof(buf)
st = State(at, at, at, at, at)
params = ctypes.create_string_buffer(%r)
def noalloc():
    n_out = ctypes.c_int64(-1)
    rc = lib.linprim_densify_noalloc(0, 0, ctypes.c_int64(8), ctypes.byref(st), buf, buf, buf, buf,
                                     params, ctypes.byref(st), ctypes.c_int64(24),
                                     ctypes.byref(n_out), None)
    assert rc == OK and n_out.value == 0, (rc, n_out.value)
noalloc()
assert get("fake_host_mallocs") == 0 and get("fake_copies") == 1
n = ctypes.c_int64(-1)
assert lib.linprim_pair_count(buf, ctypes.byref(n), None) == OK and n.value == 0
assert get("fake_host_mallocs") == 1
noalloc()
assert get("fake_host_mallocs") == 1 and get("fake_copies") == 2
""" % bytes(L.densify_params(10.0)))


def test_slot_of_a_queued_kernel_is_not_given_away(run):
    """An unrelated error on the thread while a count's kernel is queued: a
    second count that begins before the first one ends takes another slot."""
    run("""
a, b = (ctypes.c_uint64 * 8)(123), (ctypes.c_uint64 * 8)(456)
got = []
def count(x):
    n = ctypes.c_int64(-1)
    assert lib.linprim_pair_count(x, ctypes.byref(n), None) == OK
    got.append(n.value)
inside = ctypes.CFUNCTYPE(None)(lambda: count(b))
ctypes.c_int.in_dll(fake, "fake_pending_error").value = 101
ctypes.c_void_p.in_dll(fake, "fake_on_copy").value = ctypes.cast(inside, ctypes.c_void_p).value
count(a)
count(b)
assert got[-1] == 456 and 123 in got, got
assert get("fake_slots_shared") == 0
assert get("fake_pending_error") == 101
""")
