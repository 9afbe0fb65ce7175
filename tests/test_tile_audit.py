"""The tiles of the direct form and of the batched kernel audited on the CPU (no
GPU): a host driver (tests/audit/tile_audit.cpp) is compiled against the header
the kernels take their geometry and address functions from
(paper_2609_06449_amd/csrc/tile_addr.h) and enumerates every launch that the
splits of N allow, single (FP32 and split MFMA) and batched in both queue modes:
exchange buffers, items of x, ws and y, factor tables, 32-bit indexes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tiles(tmp_path):
    cc = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)
    if cc is None:
        pytest.skip("clang++ not available")
    exe = str(tmp_path / "tile_audit")
    r = subprocess.run([cc, "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2609_06449_amd", "csrc"),
                        os.path.join(ROOT, "tests", "audit", "tile_audit.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "tile audit passed" in r.stdout and "direct 2^12 x 2^11 " in r.stdout
    assert "batch, shared queue 2^10 x 2^10 " in r.stdout
