"""Operators whose slices are stencils (lists of offsets with one value each,
or with a value per row) against the same operator in its stored-entry form
(index_bytes fixed), bit for bit: the stencil form keeps the values and the
order of summation of every row, so no tolerance is needed."""

import numpy as np
import pytest
import scipy.sparse as sp

from synth import start_block
from synth.grids import grid_problem, jittered_problem
from synth.horn import horn_pencil

pytestmark = pytest.mark.gpu


def _band(n, offsets):
    """Symmetric constant-band matrix: value 1/(1+o) at offset +-o, diagonal
    dominant; offsets past the matrix are dropped."""
    offs = [o for o in offsets if 0 < o < n]
    diags = [np.full(n, 4.0)] + [np.full(n - o, -1.0 / (1 + o)) for o in offs] * 2
    return sp.csr_matrix(sp.diags(diags, [0] + offs + [-o for o in offs], shape=(n, n), format="csr"))


def _matrix(kind):
    if kind.startswith("grid"):
        S, m, _ = grid_problem(int(kind[4]), int(kind[6:]))
        return S, m
    if kind.startswith("jitter"):  # linear triangles / tetrahedra: 7 / 15 offsets, a value per row
        return jittered_problem(int(kind[6]), int(kind[8:]), 0.2, 3)
    if kind == "horn":
        return horn_pencil(5, 9, 0.05, 2)
    if kind == "broken":  # one row of one slice has a value of its own
        S = _band(200, [1, 9])
        S[70, 70] = 5.0
        return S, np.full(200, 0.5)
    if kind == "mass":  # uneven row scaling
        S = _band(200, [1, 9])
        return S, np.linspace(0.5, 1.0, 200)
    n, k = (int(v) for v in kind.split("x"))
    return _band(n, list(range(1, k + 1))), np.full(n, 0.5)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 2, 3, 8, 16])
@pytest.mark.parametrize(
    "kind",
    # rows x neighbours on one side: slice widths 1, 3, 5, 7 (the unrolled
    # lengths), 9, 31 and 33 (one past the longest stencil); less than a
    # slice, one slice, one row more, several
    ["1x1", "63x1", "64x2", "65x3", "130x4", "200x15", "200x16", "grid2_23", "grid3_9", "broken", "mass",
     "jitter2_7", "jitter2_20", "jitter3_3", "jitter3_9", "horn"],
)
def test_stencil_slices_match_stored_entries_bitwise(kind, b, precision):
    import torch

    from paper_2402_08515_amd import kf

    print(f"case stencil kind={kind} b={b} {precision}", flush=True)
    S, m = _matrix(kind)
    n = S.shape[0]
    lam = np.abs(S).sum(1).max() / m.min()
    tau = 1.8 / np.sqrt(lam)
    x = torch.from_numpy(start_block(n, b, 7)).cuda()
    for L in (2, 3, 8):  # first = last step, one middle step, steps with and without the sum
        out = []
        for ib in (0, 4):
            P = kf.Problem(S, m, 0.3 / tau, 0.6 / tau, tau, L, precision=precision, index_bytes=ib)
            out.append(P.apply_filter(x))
        assert torch.equal(out[0], out[1]), (L, (out[0] - out[1]).abs().max())


@pytest.mark.parametrize("lpr", [1, 2, 4])
@pytest.mark.parametrize("b", [2, 4, 16])
def test_stencil_lanes_per_row_bitwise(b, lpr):
    import torch

    from paper_2402_08515_amd import kf

    S, m, _ = grid_problem(3, 11)
    tau = 1.8 / np.sqrt(12.0 * 11 * 11)
    x = torch.from_numpy(start_block(S.shape[0], b, 8)).cuda()
    for precision in ("fp64", "mixed"):
        out = [kf.Problem(S, m, 4.0, 8.0, tau, 7, precision=precision, index_bytes=ib, lanes_per_row=lpr).apply_filter(x)
               for ib in (0, 2)]
        assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 2, 16])
def test_stencil_one_step_per_launch_bitwise(b, precision):
    """A cube whose band is too wide for several steps per launch."""
    import torch

    from paper_2402_08515_amd import kf

    S, m, _ = grid_problem(3, 48)
    tau = 1.8 / np.sqrt(12.0 * 48 * 48)
    x = torch.from_numpy(start_block(S.shape[0], b, 9)).cuda()
    for L in (2, 3, 8):
        out = [kf.Problem(S, m, 8.0, 16.0, tau, L, precision=precision, index_bytes=ib).apply_filter(x) for ib in (0, 4)]
        assert torch.equal(out[0], out[1]), L


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 2, 3, 8])
@pytest.mark.parametrize(
    "dim,n",
    # one slice; one workgroup with few and many slices per wavefront; several
    # workgroups with halos of one, a few and many slices (ragged last ones)
    [(2, 5), (2, 33), (2, 64), (2, 91), (2, 140), (2, 257), (3, 5), (3, 17), (3, 20), (3, 27), (3, 34)],
)
def test_several_steps_per_launch_bitwise(dim, n, b, precision):
    """The library's own choice of several steps per launch (and the
    allocation-free entry point, which has fewer buffers) against one step per
    launch: the same operations in the same order."""
    import torch

    from paper_2402_08515_amd import kf

    print(f"case steps dim={dim} n={n} b={b} {precision}", flush=True)
    S, m, _ = grid_problem(dim, n)
    tau = 1.8 / np.sqrt(4.0 * dim * n * n)
    x = torch.from_numpy(start_block(S.shape[0], b, 11)).cuda()
    for L in (3, 24, 65, 130):  # one launch, several, exactly 64 steps, a remainder after 128
        out = []
        for ib in (0, 4):
            P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, L, precision=precision, index_bytes=ib)
            out.append(P.apply_filter(x))
            if ib == 0:
                y = torch.empty_like(x)
                P.apply_filter_noalloc(x, y)
                assert torch.equal(y, out[0]), L
        assert torch.equal(out[0], out[1]), (L, (out[0] - out[1]).abs().max())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["63x1", "65x3", "200x15", "grid2_23", "grid3_9", "broken", "jitter2_20", "jitter3_9"])
def test_fourth_order_step_over_stencils_bitwise(kind, precision):
    import torch

    from paper_2402_08515_amd import kf

    S, m = _matrix(kind)
    tau = 1.8 / np.sqrt(np.abs(S).sum(1).max() / m.min())
    for b in (1, 3, 8, 16):
        x = torch.from_numpy(start_block(S.shape[0], b, 12)).cuda()
        for L in (2, 3, 8):
            out = [kf.Problem(S, m, 0.3 / tau, 0.6 / tau, tau, L, precision=precision, index_bytes=ib, stepper=4)
                   .apply_filter(x) for ib in (0, 4)]
            assert torch.equal(out[0], out[1]), (b, L)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 2, 3, 16])
@pytest.mark.parametrize(
    "kind",
    # 7 and 15 offsets with row values: less than a slice, one workgroup, few
    # and many halo slices, and (the last two) too wide a band for it
    ["jitter2_6", "jitter2_30", "jitter2_120", "jitter3_3", "jitter3_8", "jitter3_14", "horn5x40", "horn8x60", "horn16x30",
     "jitter3_24"],
)
def test_several_steps_per_launch_with_row_values_bitwise(kind, b, precision):
    import torch

    from paper_2402_08515_amd import kf

    print(f"case row-value steps kind={kind} b={b} {precision}", flush=True)
    S, m = horn_pencil(*(int(v) for v in kind[4:].split("x")), 0.05, 2) if kind.startswith("horn") else _matrix(kind)
    tau = 1.8 / np.sqrt((np.abs(S).sum(1).A1 / m).max())
    x = torch.from_numpy(start_block(S.shape[0], b, 13)).cuda()
    for L in (3, 24, 130):
        out = []
        for ib in (0, 4):
            P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, L, precision=precision, index_bytes=ib)
            out.append(P.apply_filter(x))
            if ib == 0:
                y = torch.empty_like(x)
                P.apply_filter_noalloc(x, y)
                assert torch.equal(y, out[0]), L
        assert torch.equal(out[0], out[1]), (L, (out[0] - out[1]).abs().max())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 3, 4, 16])
@pytest.mark.parametrize(
    "kind",
    # one workgroup; several with halos of one, a few and many slices; a value
    # per row with 7 and 15 offsets
    ["grid2_5", "grid2_33", "grid2_64", "grid2_140", "grid2_257", "grid3_9", "grid3_20", "grid3_27", "jitter2_40",
     "jitter3_9", "horn"],
)
def test_several_fourth_order_steps_per_launch_bitwise(kind, b, precision):
    """As above for the fourth-order step, whose two products take twice the
    halo: against two launches per step over the stored entries."""
    import torch

    from paper_2402_08515_amd import kf

    print(f"case fourth-order steps {kind} b={b} {precision}", flush=True)
    S, m = _matrix(kind)
    tau = 1.8 / np.sqrt(np.abs(S).sum(1).max() / m.min())
    x = torch.from_numpy(start_block(S.shape[0], b, 13)).cuda()
    for L in (3, 24, 70):  # one launch, several, a remainder
        out = []
        for ib in (0, 4):
            P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, L, precision=precision, index_bytes=ib, stepper=4)
            out.append(P.apply_filter(x))
            if ib == 0:
                y = torch.empty_like(x)
                P.apply_filter_noalloc(x, y)
                assert torch.equal(y, out[0]), L
        assert torch.equal(out[0], out[1]), (L, (out[0] - out[1]).abs().max())
