"""Host code of the library against a stub of the HIP runtime (hip_stub.c): two
devices in host memory, kernels that do nothing.  What is allocated, where and
when; which device's handles a call uses.  Each test runs in a child process
that loads the stub before the library.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_0710_5912_amd", "libmodelh.so")

HEAD = """
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stub.stub_used.restype = C.c_size_t
stub.stub_mallocs.restype = stub.stub_events.restype = stub.stub_launches.restype = C.c_long
stub.stub_limit.argtypes = [C.c_size_t]
lib = C.CDLL(sys.argv[2])
used = lambda: [stub.stub_used(d) for d in range(2)]
def net(h, w):
    p = C.c_void_p()
    assert lib.le_cnn_create(h, w, C.byref(p)) == 0
    return p
def grad(p, batch, h, w):
    x = (C.c_float * (2 * h * w * batch))()
    loss = C.c_double()
    return lib.le_cnn_grad(p, x, x, batch, C.byref(loss), None, None)
def context(nx, ny):
    sys.path.insert(0, ".")
    from paper_0710_5912_amd import le
    p = le.make_params(dict(nx=nx, ny=ny, lx=float(nx), ly=float(ny), gdot=0.01, A=1.0, B=1.0,
                            kappa=1.0, M=1.0, eta=1.0, rho=1.0, dt=0.005))
    c = C.c_void_p()
    assert lib.le_create(C.byref(p), (C.c_double * (nx * ny))(), None, C.byref(c)) == 0
    return c
def tuning(c):
    t = (C.c_int32 * 10)()
    assert lib.le_tuning(c, t, 10) == 1
    return list(t)
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    cc = shutil.which("gcc")
    if cc is None or not os.path.exists(LIB):
        pytest.skip("no host compiler, or the library is not built")
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-pthread", "-o", out,
                    os.path.join(ROOT, "tests", "hip_stub.c")], check=True)
    return out


def child(stub, body):
    r = subprocess.run([sys.executable, "-c", HEAD + body, stub, LIB], capture_output=True,
                       text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr


def test_training_workspace_is_on_the_networks_device(stub):
    child(stub, """
stub.hipSetDevice(1)
n = net(32, 32)
before = used()
stub.hipSetDevice(0)
assert grad(n, 8, 32, 32) == 0
dev = C.c_int()
stub.hipGetDevice(C.byref(dev))
assert dev.value == 0
assert used()[0] == 0 and used()[1] > before[1], used()
lib.le_cnn_destroy(n)
assert used() == [0, 0], used()
""")


@pytest.mark.parametrize("h,w", [(16, 16), (64, 32), (256, 256), (1024, 1024)])
def test_training_network_holds_one_samples_buffers(stub, h, w):
    """844 bytes per pixel (activations, pre-activations, two gradients) and 144 for
    the weight gradient's partials, what one layer's take; 2 MB for the rest."""
    child(stub, f"""
n = net({h}, {w})
assert used()[0] <= (844 + 144) * {h * w} + (2 << 20), used()
""")


def test_training_workspace_settles_where_memory_is_short(stub):
    """16 samples of 64^2 do not fit, 8 do: they are taken once and kept."""
    child(stub, """
n = net(64, 64)
stub.stub_limit(used()[0] + 12 * 900 * 64 * 64)
assert grad(n, 16, 64, 64) == 0
held, calls = used(), stub.stub_mallocs()
assert held[0] > 8 * 844 * 64 * 64
assert grad(n, 16, 64, 64) == 0 and grad(n, 16, 64, 64) == 0
assert used() == held and stub.stub_mallocs() == calls
stub.stub_limit(1 << 62)
assert grad(n, 32, 64, 64) == 0 and used()[0] > 32 * 844 * 64 * 64
lib.le_cnn_destroy(n)
assert used() == [0, 0]
""")


def test_large_fields_are_read_back_from_any_threads_device(stub):
    """A context of device 1 read by a thread whose current device is 0: what the
    call waits on belongs to the context's device."""
    child(stub, """
import threading
phi = (C.c_double * (1024 * 512))()
rc = []
stub.hipSetDevice(1)
c = context(1024, 512)
read = lambda: rc.append(lib.le_get_state(c, phi, phi, phi, None, None))   # a new thread: device 0
t = threading.Thread(target=read)
t.start()
t.join()
assert rc == [0], rc
lib.le_destroy(c)
""")


def test_tuning_file_of_other_shapes_is_passed_over(stub, tmp_path):
    """A line as a library with other column shapes wrote it (device, grid, precision,
    inertia, runs; six variants) leaves the choice alone; a written one is found."""
    f = tmp_path / "tune"
    f.write_text("0 64 64 0 1 1 33 33 4 4 5 5\n")
    for _ in range(2):
        child(stub, f"""
import os
os.environ["LE_TUNE_CACHE"] = {str(f)!r}
assert tuning(context(64, 64))[4:] == [0, 0, 0, 0, 0, 0]
""")
    lines = [list(map(int, line.split())) for line in f.read_text().splitlines()]
    assert len(lines) == 2 and lines[1][1:] == [64, 64, 0, 1, 1, 0, 0, 0, 0, 0, 0]


def test_only_stages_that_a_step_runs_are_timed(stub):
    """6 + 6 row, 5 + 5 column candidates, each launched 1 + 9 times, the inverse rows
    two kernels at a time; where the stages are apart also 21 + 18 stencil ones."""
    child(stub, """
import os
launched = lambda: (context(64, 64), stub.stub_launches())[1]
setup = 50
joined = launched()
assert joined <= 10 * (12 + 6 + 5 + 5) + setup, joined
assert launched() <= joined + setup            # found in the cache
at = stub.stub_launches()
os.environ["LE_TUNE_ROW"] = "0"                # apart: an entry of its own
assert launched() - at >= 10 * (6 + 5 + 5 + 21 + 18)
""")
