"""Tree selection in rounds, its device function run on the host.

tests/native/tree_rounds_check.cpp compiles tree_rounds.hpp for the host and
runs it with a workgroup's threads as fibers, for all three row tables: what it
finishes equals a walk that pops one node at a time, and it finishes what it
is meant to (on the GPU a selection that handed everything over would give the
same trees).
"""
import os
import subprocess

import pytest

from paper_2606_03819_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rounds_on_the_host(tmp_path):
    hipcc = build.hipcc()
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = tmp_path / "tree_rounds_check"
    src = os.path.join(HERE, "native", "tree_rounds_check.cpp")
    inc = os.path.join(os.path.dirname(HERE), "paper_2606_03819_amd", "csrc")
    rocm_inc = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "include")
    c = subprocess.run([hipcc, "-O1", "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", rocm_inc, "-I", inc,
                        src, "-o", str(exe)], capture_output=True, text=True)
    assert c.returncode == 0, c.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
    assert r.stdout.strip().endswith(" 0 failures")
