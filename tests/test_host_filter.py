"""Step buffers and recordings of the filter applications, on the CPU: the
library's host code (kf_api.cpp) compiled against a runtime that keeps books of
device memory, recordings and launches (host_filter.cpp)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(INCLUDE, "hip")):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("host") / "host_filter")
    cmd = ["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", INCLUDE,
           os.path.join(HERE, "host_filter.cpp"), "-o", out, "-lpthread",
           # the parts of the library that no scenario reaches
           "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def _run(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize(
    "scenario", ["alternate2", "alternate4", "wide_then_recorded", "no_second_pair_1", "no_second_pair_2"]
)
def test_step_buffers(program, scenario):
    _run(program, scenario)


def test_recordings_of_alternating_widths(program):
    _run(program, "chunks")


def test_block_widths_of_a_batch(program):
    _run(program, "batch_widths")
