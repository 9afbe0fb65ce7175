"""Host code under failed device allocations, on the CPU: the library is loaded
against a stub of the HIP runtime (tests/stub/hip_stub.c) in a process of its
own, which fails the allocations that a case names."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2609_06449_amd import paco

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1])
hip.stub_fail_mallocs.argtypes = [ctypes.c_uint64]
from paper_2609_06449_amd import paco
IN, OUT, WS = 1 << 40, 1 << 41, 1 << 42   # never read: launches do nothing


def plan(shape, fail):
    hip.stub_fail_mallocs(fail)
    assert hip.hipPeekAtLastError() == 0
    p = paco.Plan(*shape, 64, 4)
    assert hip.hipPeekAtLastError() == 0, "an error left behind by a plan that was made"
    return p


def runs(p, launches, inverse=True):
    n = hip.stub_launches()
    p.execute(IN, OUT, WS)
    assert hip.stub_launches() - n == launches == p.launches, (hip.stub_launches() - n, p.launches)
    if inverse:
        p.execute_inverse(IN, OUT, WS)


def closed(p):
    p.close()
    assert hip.stub_mallocs() == hip.stub_frees(), (hip.stub_mallocs(), hip.stub_frees())


# 16384 x 16384: the second allocation is the balanced shape's, which paco_execute runs
p = plan((1 << 14, 1 << 14), 0)
assert hip.stub_mallocs() == 2 and "executes" in p.description
runs(p, 3); closed(p)
p = plan((1 << 14, 1 << 14), 2)
assert hip.stub_mallocs() == 2 and "executes" not in p.description and p.has_split == 2
runs(p, 3); closed(p)
# 1024 x 16384: without the balanced shape its own passes, forward and inverse
p = plan((1 << 10, 1 << 14), 2)
assert hip.stub_mallocs() == 3 and "executes" not in p.description
runs(p, p.launches); closed(p)
# 16384 x 4096: the second allocation is the inverse's; without any the forward transform stands
p = plan((1 << 14, 1 << 12), 2)
assert hip.stub_mallocs() == 3
runs(p, 3); closed(p)
p = plan((1 << 14, 1 << 12), 6)
runs(p, 3, inverse=False)
try:
    p.execute_inverse(IN, OUT, WS)
    raise SystemExit("the inverse ran without passes")
except paco.PacoError as e:
    assert e.status == paco.PACO_ERR_UNSUPPORTED and "out of memory" in str(e), e
runs(p, 3, inverse=False); closed(p)
# no memory for the plan itself, nor for a batch plan: the status says so, and nothing else does
for make in (lambda: paco.Plan(64, 64, 4, 4), lambda: paco.Plan(1 << 14, 1 << 14, 64, 4),
             lambda: paco.BatchPlan([64] * 3), lambda: paco.BatchPlan([1 << 17] * 3)):
    hip.stub_fail_mallocs(1)
    try:
        make()
        raise SystemExit("a plan without memory")
    except paco.PacoError as e:
        assert e.status == paco.PACO_ERR_ALLOC, e
    assert hip.hipPeekAtLastError() == 0
    assert hip.stub_mallocs() == hip.stub_frees()
print("ok")
"""


def test_failed_allocations_leave_no_error_and_no_memory_behind(tmp_path):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    stub = str(tmp_path / "libamdhip64.so.7")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-Wall", os.path.join(ROOT, "tests", "stub", "hip_stub.c"), "-o", stub,
                    "-Wl,-soname,libamdhip64.so.7"], check=True)
    assert paco.lib() is not None
    env = dict(os.environ, LD_LIBRARY_PATH=str(tmp_path))
    r = subprocess.run([sys.executable, "-c", SCRIPT, stub], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
