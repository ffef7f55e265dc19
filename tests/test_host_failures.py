"""Host code of the library where the runtime refuses an allocation, against a
stand-in for the HIP runtime (hip_stub.c): no device, kernels do nothing, so
graphs here have no edges. Each test runs in a process of its own, where the
stand-in is loaded under the runtime's name before the library."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.modules["torch"] = None  # torch would bring the real runtime
sys.path.insert(0, {root!r})
stub = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
for f in ("stub_host_allocs", "stub_pool_idle", "stub_trims"):
    getattr(stub, f).restype = ctypes.c_int64
for f in ("stub_fail_host", "stub_device_limit"):
    getattr(stub, f).argtypes = [ctypes.c_int64]
import numpy as np
from paper_2009_10955_amd import gp
from paper_2009_10955_amd import inputs as I
def edgeless(n=5):
    return gp.Graph(np.zeros(n + 1, np.int64), np.zeros(0, np.int32), stream=0)
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "libamdhip64.so.7")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wl,-soname,libamdhip64.so.7", "-o", out,
                    os.path.join(HERE, "hip_stub.c")], check=True)
    return out


def _run(stub, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, stub=stub) + body], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_count_without_a_pinned_page(stub):
    """The page that results are written to cannot be had: the call copies its
    result instead, and the refused allocation is not reported as a launch's error."""
    _run(stub, """
g = edgeless()
plan = gp.Plan(*I.PATTERNS["4-cycle"])
stub.stub_fail_host(1000)
assert gp.count(g, plan, stream=0) == 0
assert gp.count(g, plan, stream=0) == 0
stub.stub_fail_host(0)
assert gp.count(g, plan, stream=0) == 0 and stub.stub_host_allocs() == 1
""")


def test_graphs_share_one_pinned_page(stub):
    """Loading, counting and freeing graphs one after another pins memory once."""
    _run(stub, """
for n in (3, 5, 9):
    g = edgeless(n)
    assert gp.count(g, gp.Plan(*I.PATTERNS["edge"]), stream=0) == 0
    g.close()
assert stub.stub_host_allocs() == 1, stub.stub_host_allocs()
""")


def test_idle_pool_memory_is_given_back_to_a_refused_allocation(stub):
    """Memory that the calls' pool holds idle does not fail a load: the pool is
    trimmed and the allocation tried again."""
    _run(stub, """
g = edgeless()
assert gp.check_sum(np.ones(1 << 20, np.uint64), stream=0) is not None
idle = stub.stub_pool_idle()
assert idle >= 8 << 20
stub.stub_device_limit(idle + (4 << 20))
big = edgeless((1 << 20) - 1)  # 8 MB of row pointers
assert stub.stub_trims() == 1 and stub.stub_pool_idle() < idle
big.close()
g.close()
""")


def test_refused_scratch_leaves_no_error_behind(stub):
    """A count whose scratch is refused returns GP_ERR_NOMEM, and the next one, with
    memory there again, counts."""
    _run(stub, """
g = edgeless()
plan = gp.Plan(*I.PATTERNS["4-cycle"])
stub.stub_device_limit(1)
try:
    gp.count(g, plan, stream=0)
    raise SystemExit("not refused")
except gp.GpError as e:
    assert e.status == -7, e
stub.stub_device_limit(0)
assert gp.count(g, plan, stream=0) == 0
""")


def test_pool_is_not_used_while_no_graph_is_loaded(stub):
    """Nothing would give the pool's memory back then."""
    _run(stub, """
gp.check_sum(np.ones(1 << 20, np.uint64), stream=0)
assert stub.stub_pool_idle() == 0
""")
