"""The library's host path under failures that a GPU does not produce on demand: the library runs in a process of its own on
tests/host/fake_hip.cpp, a HIP runtime that runs nothing, writes down what it is asked for and fails where it is told to."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

from paper_2309_15531_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PREAMBLE = """
import ctypes, sys
from ctypes import byref, c_int32, c_int64, c_void_p, c_char_p, c_double
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # ahead of the HIP runtime the library is linked with
fake.fake_calls.restype = c_char_p
lib = ctypes.CDLL(sys.argv[2])
lib.adadim_last_error.restype = c_char_p
OK, EHIP, EINVAL = %d, %d, %d
def context(stream=0x1000):
    h = c_void_p()
    assert lib.adadim_create(byref(h), c_void_p(stream)) == OK
    return h
def calls():
    return fake.fake_calls().decode().split("\\n")[:-1]
def launched(name):
    return [c for c in calls() if c.startswith("launch") and name in c]
A = c_void_p(0x10000)                                          # aligned, never dereferenced: nothing runs
def gemv(ctx, out, inn, bits=4):
    return lib.adadim_gemv_ic(ctx, A, A, A, A, c_int64(out), c_int64(inn), bits, 32, A)
""" % (B.OK, B.EHIP, B.EINVAL)


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    if not os.path.exists(B.LIB_PATH):
        from paper_2309_15531_amd.build import build
        build(verbose=False)
    fake = tmp_path_factory.mktemp("fake") / "libfake_hip.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "host", "fake_hip.cpp"), "-o",
                    str(fake)], check=True)

    def go(body):
        res = subprocess.run([sys.executable, "-c", PREAMBLE + textwrap.dedent(body), str(fake), B.LIB_PATH],
                             capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stdout + res.stderr
        return res.stdout
    return go


def test_a_failed_allocation_fails_no_later_call(run):
    """The runtime keeps the error of a failed allocation until it is asked for; the next call's launches must not report it."""
    run("""
    ctx = context()
    for call in (lambda: gemv(ctx, 4096, 4096), lambda: lib.adadim_select(ctx, A, 2, None, byref(c_int32()))):
        fake.fake_reset()
        fake.fake_fail(b"hipMalloc", 1)
        assert call() == EHIP
        assert call() == OK, lib.adadim_last_error(ctx)
    """)
