"""The filter-weight network pins host memory for its first gradient, not when
it is made, on the CPU (host_network.cpp)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_memory_is_pinned_for_the_first_gradient(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path / "host_network")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-nogpulib", "-std=c++17", "-w",
           os.path.join(HERE, "host_network.cpp"), "-o", out, "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
