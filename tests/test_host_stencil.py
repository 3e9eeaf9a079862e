"""The build of an operator's stencil form when the device has no memory for
it, on the CPU: the form is left out, and the operator keeps its stored
entries (host_stencil.cpp)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_memory_for_the_stencil_form(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path / "host_stencil")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-nogpulib", "-std=c++17", "-w",
           os.path.join(HERE, "host_stencil.cpp"), "-o", out, "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
