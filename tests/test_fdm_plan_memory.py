"""Failing allocations while the fast-diagonalisation plan is built, its threads included
(tests/host/fdm_plan_memory_check.cpp, on the CPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_plan_survives_failing_allocations(tmp_path):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "fdm_plan_memory_check")
    src = os.path.join(ROOT, "paper_2505_16992_amd", "csrc")
    cmd = [cxx, "-std=c++17", "-O2", "-pthread", "-I" + os.path.join(ROOT, "include"),
           os.path.join(HERE, "host", "fdm_plan_memory_check.cpp"), os.path.join(src, "piso_fdm_plan.cpp"),
           os.path.join(src, "piso_topology.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, (r.stdout + r.stderr)[-2000:])
