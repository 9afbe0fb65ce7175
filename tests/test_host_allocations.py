"""The library's host code and its device allocations, on the CPU: the library is
loaded against a stub of the HIP runtime (tests/stub/hip_stub.c) in a process of
its own, which counts allocations and fails those that a case names."""
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

TABLES = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1])
hip.stub_bytes.restype = ctypes.c_uint64
hip.stub_fail_mallocs.argtypes = [ctypes.c_uint64]
from paper_2609_06449_amd import paco


def tables(shape, **kw):
    hip.stub_fail_mallocs(0)
    p = paco.Plan(*shape, 2, 2, **kw)
    return p.description, hip.stub_bytes()


for shape in ((256, 256), (1024, 512), (1024, 1024), (2048, 1024), (2048, 2048)):
    (direct, a), (phases, b) = tables(shape), tables(shape, flags=paco.PACO_PLAN_NO_SPLIT)
    assert " direct[two column passes, " in direct and " direct[" not in phases
    assert a == b if shape[0] == shape[1] else a < b, (shape, a, b)  # (b: with the swapped shape's for the inverse)

# the balanced shape behind a plan: its symmetric passes only, not the tables of
# Phase II's hook (128 x 128) and of the two-pass form (16 x 4096)
hip.stub_size.restype = ctypes.c_uint64
assert "executes sym[" in tables((1 << 10, 1 << 14))[0]
second = hip.stub_size(1)
assert "executes" not in tables((1 << 12, 1 << 12))[0]
assert second == hip.stub_size(0) - 8 * (128 * 128 + 16 * 4096), (second, hip.stub_size(0))
print("ok")
"""


def _on_the_stub(tmp_path, script):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    stub = str(tmp_path / "libamdhip64.so.7")
    subprocess.run([cc, "-O1", "-shared", "-fPIC", "-Wall", os.path.join(ROOT, "tests", "stub", "hip_stub.c"), "-o", stub,
                    "-Wl,-soname,libamdhip64.so.7"], check=True)
    assert paco.lib() is not None
    env = dict(os.environ, LD_LIBRARY_PATH=str(tmp_path))
    r = subprocess.run([sys.executable, "-c", script, stub], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


def test_failed_allocations_leave_no_error_and_no_memory_behind(tmp_path):
    _on_the_stub(tmp_path, SCRIPT)


def test_column_passes_take_no_second_table(tmp_path):
    # w_{16 N1}^{-k} is the two-pass form's table as well
    _on_the_stub(tmp_path, TABLES)
