"""Error paths of the library with HIP calls that fail where a test says so (tests/hip_failures.c).  Each case runs in a process
of its own, since the library must find the failing calls before the runtime's."""
import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
PROLOGUE = """
import ctypes as C, sys
sys.path.insert(0, %r)
shim = C.CDLL(%r, mode=C.RTLD_GLOBAL)
import numpy as np
from paper_2204_07104_amd import binding
assert shim.hip_failures_runtime(binding.hip_runtime_path().encode())
rng = np.random.default_rng(1)
dims, J, R = (70_001, 311), (61, 33), 40
idx = [rng.integers(0, d, 2_000).astype(np.int32) for d in dims]
A = [rng.standard_normal((d, j)).astype(np.float32) for d, j in zip(dims, J)]
B = [rng.standard_normal((j, R)).astype(np.float32) for j in J]
ft = binding.FastTucker(dims, idx, np.ones(2_000, dtype=np.float32), J, R)
def refused(call, code):
    try:
        call()
    except binding.FtkError as e:
        assert e.code == code, e
        return
    raise AssertionError("no error")
def same(got, want):
    assert all(np.array_equal(x, y) for x, y in zip(sum(got, []), sum(want, [])))
"""


def run(tmp_path, body):
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no gcc")
    shim = str(tmp_path / "hip_failures.so")
    subprocess.check_call([gcc, "-shared", "-fPIC", "-O1", "-Wall", "-Werror", os.path.join(HERE, "hip_failures.c"), "-o", shim, "-ldl"])
    done = subprocess.run([sys.executable, "-c", PROLOGUE % (os.path.dirname(HERE), shim) + body], capture_output=True, text=True, timeout=90)
    print(done.stdout, done.stderr, flush=True)
    assert done.returncode == 0


def test_factors_move_after_an_event_could_not_be_made(tmp_path):
    """The first transfer makes the events of its ring; one that cannot be made fails that call only."""
    run(tmp_path, """
for k in (1, 3):
    shim.hip_failures_set(k, 0)
    refused(lambda: ft.ftk_set_factors(A, B), binding.FTK_ENOMEM)
    shim.hip_failures_set(0, 0)
ft.ftk_set_factors(A, B)
same(ft.ftk_get_factors(), (A, B))
""")


def test_a_transfer_that_fails_half_way_leaves_nothing_in_the_stream(tmp_path):
    """The chunks under way are waited for before the call returns: the ring is the next call's, and a held-out set's records are
    freed."""
    run(tmp_path, """
hip = C.CDLL(binding.hip_runtime_path())
held = [rng.integers(0, d, 1_500_000).astype(np.int32) for d in dims], np.ones(1_500_000, dtype=np.float32)
ft.ftk_set_factors(A, B)
want = ft.ftk_evaluate(*held)
calls = (lambda: ft.ftk_set_factors([2 * a for a in A], B), lambda: ft.ftk_get_factors(), lambda: ft.ftk_evaluate(*held))
for call in calls:
    for k in (1, 3, 5):      # (17 and 18 MB: five chunks of up to 4 MB each)
        shim.hip_failures_set(0, k)
        refused(call, binding.FTK_EDEVICE)
        assert hip.hipStreamQuery(None) == 0
        shim.hip_failures_set(0, 0)
        ft.ftk_set_factors(A, B)
        same(ft.ftk_get_factors(), (A, B))
assert np.allclose(ft.ftk_evaluate(*held), want, rtol=1e-12)
""")
