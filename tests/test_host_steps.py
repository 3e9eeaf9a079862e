"""Which operators take several steps per launch, by the library's own rule, on
the CPU (host_steps.cpp).  The GPU tests of those kernels compare results that
every path gives, so the meshes they use are held here to the path they are
meant for, and others to one step per launch."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from synth.grids import grid_problem, jittered_problem
from synth.horn import horn_pencil

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("host") / "host_steps")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-nogpulib", "-std=c++17", "-w",
           os.path.join(HERE, "host_steps.cpp"), "-o", out, "-Wl,--unresolved-symbols=ignore-all"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def ask(line):
        r = subprocess.run([out], input=line + "\n", capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, r.stderr
        return [int(v) for v in r.stdout.split()]

    return ask


def _operator(kind):
    """rows, largest offset, entries of the longest list and as stored, value per row"""
    mesh, size = kind.split("_")
    if mesh == "horn":
        S = horn_pencil(*(int(v) for v in size.split("x")), 0.05, 2)[0]
    elif mesh.startswith("jitter"):
        S = jittered_problem(int(mesh[-1]), int(size), 0.2, 3)[0]
    else:
        S = grid_problem(int(mesh[-1]), int(size))[0]
    row = np.repeat(np.arange(S.shape[0]), np.diff(S.indptr))
    lists = np.unique(np.stack([row // 64, S.indices - row]), axis=1)
    width, row_values = int(np.bincount(lists[0]).max()), not mesh.startswith("grid")
    stored = width if width in ((15,) if row_values else (5, 7)) else (width + 3) // 4 * 4
    return S.shape[0], int(np.abs(lists[1]).max()), width, stored, int(row_values)


def _steps(rule, kind, b, value_bytes, L, order, replay=1):
    return rule("one " + " ".join(str(v) for v in (*_operator(kind), value_bytes, b, L, int(order == 4), replay)))[0]


@pytest.mark.parametrize("value_bytes", [4, 8])
@pytest.mark.parametrize(
    "kind,order,b",
    [("grid2_5", 2, 1), ("grid2_64", 2, 8), ("grid2_140", 2, 2), ("grid2_257", 2, 4), ("grid3_5", 2, 8), ("grid3_20", 2, 1),
     ("jitter2_6", 2, 16), ("jitter2_120", 2, 2), ("jitter3_8", 2, 16), ("horn_5x40", 2, 16), ("horn_8x60", 2, 4),
     ("grid2_33", 4, 16), ("grid2_257", 4, 4), ("grid3_9", 4, 16), ("grid3_20", 4, 1), ("jitter2_40", 4, 16),
     ("jitter3_9", 4, 16), ("horn_5x9", 4, 4)],
)
def test_several_steps_per_launch(rule, kind, order, b, value_bytes):
    assert _steps(rule, kind, b, value_bytes, 24, order) > 1


@pytest.mark.parametrize("value_bytes", [4, 8])
@pytest.mark.parametrize(
    "kind,order,b",
    [("grid3_34", 2, 1), ("grid3_48", 2, 1), ("grid3_20", 2, 16), ("jitter3_24", 2, 1), ("horn_16x30", 2, 1),
     ("horn_8x60", 2, 16), ("grid2_257", 4, 16), ("grid3_27", 4, 1)],
)
def test_one_step_per_launch(rule, kind, order, b, value_bytes):
    assert _steps(rule, kind, b, value_bytes, 24, order) == 0


def test_the_meshes_of_the_recorded_steps(rule):
    """One step per launch where it is replayed, whatever the width."""
    for kind, b, value_bytes in (("grid3_44", 1, 8), ("grid3_44", 4, 4), ("grid3_41", 4, 8), ("jitter3_26", 2, 8),
                                 ("jitter3_26", 8, 4)):
        for order in (2, 4):
            assert _steps(rule, kind, b, value_bytes, 30, order) == 0, (kind, b, order)


def test_alternating_widths_take_both_paths(rule):
    assert [_steps(rule, "grid2_300", b, 8, 40, 2) > 1 for b in (1, 2, 4, 8, 16)] == [True, True, True, False, False]


@pytest.mark.parametrize("value_bytes", [4, 8])
def test_members_of_a_batch(rule, value_bytes):
    """Small members take several steps each, side by side; not where one of
    them has too wide a band."""
    small = "2 303 139 41 8 64 66"  # a square of 140 cells, a cube of 9
    steps = rule(f"batch {value_bytes} 1 {small}")
    assert len(steps) == 2 and min(steps) > 1
    assert rule(f"batch {value_bytes} 1 1 2073 2601 40") == []  # a cube of 52 cells
