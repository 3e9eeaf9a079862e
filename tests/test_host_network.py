"""The filter-weight network's host memory, on the CPU (host_network.cpp): it is
pinned for the first gradient, not when the network is made, and a training
run's losses come back through a bounded block."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("host") / "host_network")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-nogpulib", "-std=c++17", "-w",
           os.path.join(HERE, "host_network.cpp"), "-o", out, "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def _run(program, *args):
    r = subprocess.run([program, *args], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_memory_is_pinned_for_the_first_gradient(program):
    _run(program)


def test_losses_of_a_long_run(program):
    _run(program, "long")
