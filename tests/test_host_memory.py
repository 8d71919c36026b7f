"""Device memory as the library's host side asks for it, on the CPU: libcwo.so bound to a runtime
that only counts allocations (stub_runtime.cpp), each case in a process of its own. What is
checked are return codes and bytes; no kernel runs."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_held.restype = ctypes.c_size_t
stub.stub_refuse.argtypes = [ctypes.c_size_t]
from paper_1107_5578_amd import cwo
lib = cwo.load()
PTR = ctypes.c_void_p(1 << 20)  # the caller's device memory: never read here

class Ctx:
    def __init__(self, budget=0):
        self.h = ctypes.c_void_p()
        assert lib.cwo_create(ctypes.byref(self.h), 0, budget) == 0
    def asm(self, nx, ny, precision="f32"):
        p = cwo.make_params(nx, ny, 8e-6, precision=precision)
        return lib.cwo_asm(self.h, ctypes.byref(p), PTR, PTR, None)
    def pls(self, nx, ny, points, field=False):
        p = cwo.PlsParams(nx, ny, 4e-6, 4e-6, 633e-9, 0.0, 0.0, 0.1)
        fn = lib.cwo_pls_field if field else lib.cwo_pls_cgh
        return fn(self.h, ctypes.byref(p), PTR, points, PTR, None)
    def gs(self, nx, ny, iterations, precision="f32"):
        p = cwo.make_params(nx, ny, 8e-6, precision=precision)
        return lib.cwo_gs(self.h, ctypes.byref(p), PTR, PTR, PTR, iterations, PTR, None)
    def held(self):
        n = ctypes.c_size_t()
        assert lib.cwo_memory_held(self.h, ctypes.byref(n)) == 0
        return n.value
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "libstub_runtime.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so,
                           os.path.join(HERE, "stub_runtime.cpp")])
    return so


def run(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, stub], cwd=ROOT, timeout=120,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("call", ["c.asm(256, 256)", "c.pls(64, 64, 100)", "c.gs(256, 256, 3)"])
def test_refused_allocation_does_not_end_the_context(stub, call):
    """A device that is out of memory fails the call, not the calls after it."""
    run(stub, """
c = Ctx()
stub.stub_refuse(1)
assert %s == cwo.CWO_ERR_NOMEM
stub.stub_refuse(0)
assert %s == cwo.CWO_OK
""" % (call, call))


def test_refused_partial_sums(stub):
    """Without memory for partial sums a point-light-source call takes one range of points."""
    run(stub, """
c = Ctx()
stub.stub_refuse(64 << 20)
assert c.pls(512, 512, 4000) == cwo.CWO_OK
assert c.held() == 32 * 4000 == stub.stub_held()
stub.stub_refuse(0)
assert c.asm(256, 256) == cwo.CWO_OK
assert c.pls(512, 512, 4000) == cwo.CWO_OK
""")


@pytest.mark.parametrize("nx,ny,iterations", [(2048, 2048, 200), (256, 512, 7), (4096, 64, 5)])
@pytest.mark.parametrize("precision,elem", [("f32", 8), ("f16", 4)])
def test_gs_scratch(stub, nx, ny, iterations, precision, elem):
    """The iteration's scratch is the padded spectrum and one error partial per row and 1024
    padded points, so a budget of that size (FP16: and of the range pre-pass) is enough."""
    need = elem * ny * 2 * nx + 8 * (iterations * ny * max(1, 2 * nx // 1024) + 512)
    run(stub, """
need = %d
c = Ctx(need if %r == "f32" else need + (64 << 10))
assert c.gs(%d, %d, %d, %r) == cwo.CWO_OK
""" % (need, precision, nx, ny, iterations, precision))


@pytest.mark.parametrize("n", [64, 256, 4096])
def test_served_requests_in_a_tight_budget(stub, n):
    """A budget of one request's footprint and the roots of unity of its transforms serves one
    request after the other."""
    run(stub, """
n = %d
c = Ctx(16 * n * n + 8 * n * 2 * n + 8 * 2 * n)
for k in range(3):
    job = cwo.Job(cwo.make_params(n, n, 8e-6, kind=cwo.ANGULAR), PTR, PTR)
    t, state = ctypes.c_uint64(), ctypes.c_int32()
    assert lib.cwo_submit(c.h, ctypes.byref(job), ctypes.byref(t)) == 0
    assert lib.cwo_drain(c.h) == 0
    assert lib.cwo_poll(c.h, t.value, ctypes.byref(state)) == 0
    assert state.value == cwo.DONE, k
""" % n)


def test_partial_sums_while_another_stream_records(stub):
    """A call whose records fit may run while another stream of the process records a graph: its
    first partial sums are allocated without ending that capture."""
    run(stub, """
c = Ctx()
assert c.pls(2048, 2048, 4596) == cwo.CWO_OK
assert c.held() == 32 * 4596
stub.stub_record(1)
assert c.pls(512, 512, 4000) == cwo.CWO_OK
assert stub.stub_unsafe_allocations() == 0
assert c.held() == 32 * 4596 + (64 << 20)
""")
