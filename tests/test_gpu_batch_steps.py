"""Batched filter applications whose small members take several steps per
launch, beside the members that take one, against the stored-entry form of the
same batch (index_bytes fixed: one step per launch), bit for bit: the same
operations in the same order, so no tolerance is needed."""

import numpy as np
import pytest
import scipy.sparse as sp

from synth import start_block
from synth.grids import grid_problem, jittered_problem

pytestmark = pytest.mark.gpu

# (mesh, cells, L).  Members of one slice, of one workgroup and of several with
# halos of one and of many slices, with no step, one step, less than a launch's
# steps and several launches of them; "mixed" beside cubes too large for it,
# "small" with no other member, "uneven" with a member whose slices hold a value
# per row and "wide" with one that has more offsets than the stencil form takes,
# which both keep the batch at one step per launch (of the members in two groups),
# as lists shorter than the kernel's do ("chain", three offsets).
BATCHES = {
    "mixed": [("square", 5, 3), ("square", 64, 60), ("cube", 52, 40), ("square", 91, 33), ("square", 64, 1),
              ("square", 33, 130), ("cube", 17, 24), ("square", 64, 2), ("cube", 40, 7), ("square", 187, 90)],
    "small": [("square", 140, 41), ("cube", 9, 66)],
    "uneven": [("square", 33, 12), ("jitter", 20, 21)],
    "wide": [("square", 33, 12), ("band", 300, 21), ("square", 64, 30)],
    "chain": [("chain", 300, 33), ("chain", 64, 12)],
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("b", [1, 2, 3, 8, 16])
@pytest.mark.parametrize("name", list(BATCHES))
def test_batch_with_several_steps_per_launch_bitwise(name, b, precision):
    import torch

    from paper_2402_08515_amd import kf

    print(f"case batch steps {name} b={b} {precision}", flush=True)
    members = []
    for mesh, n, L in BATCHES[name]:
        dim = 3 if mesh == "cube" else 2
        if mesh in ("band", "chain"):  # 33 offsets, 3
            r = 16 if mesh == "band" else 1
            S = sp.csr_matrix(sp.diags([4.0] + [-0.8 / r] * (2 * r), list(range(r + 1)) + list(range(-r, 0)), shape=(n, n)))
            m = np.full(n, 0.5)
        else:
            S, m = jittered_problem(2, n, 0.2, 3) if mesh == "jitter" else grid_problem(dim, n)[:2]
        tau = 1.8 / (abs(S).sum(1).max() / m.min()) ** 0.5
        members.append((S, m, 0.3 / tau, 0.5 / tau, tau, L, 0))
    free = kf.Batch(members, precision=precision)
    fixed = kf.Batch(members, precision=precision, index_bytes=4)
    # the recorded application is replayed on new inputs, with other work between
    for rep in range(3):
        xs = [torch.from_numpy(start_block(S.shape[0], b, 10 * rep + i)).cuda()
              for i, (S, *_rest) in enumerate(members)]
        got, ref = free.apply_filter(xs), fixed.apply_filter(xs)
        for (_, n, L), y, r in zip(BATCHES[name], got, ref):
            assert torch.equal(y, r), (rep, n, L, (y - r).abs().max())
        torch.ones(1 << 20, device="cuda").sum().item()


@pytest.mark.parametrize("b", [1, 3, 4])
def test_column_major_blocks_equal_row_major_ones(b):
    """The two layouts of a batch's blocks (members with no step, one step and
    several, stored entries too): only the addresses differ."""
    import ctypes as C

    import torch

    from paper_2402_08515_amd import kf

    print(f"case batch layouts b={b}", flush=True)
    for options in ({}, {"index_bytes": 4}):
        members = []
        for n, L in ((20, 1), (33, 2), (90, 23)):
            S, m = grid_problem(2, n)[:2]
            tau = 1.8 / (8.0 * n * n) ** 0.5
            members.append((S, m, 0.3 / tau, 0.5 / tau, tau, L, 0))
        bt = kf.Batch(members, **options)
        xs = [torch.from_numpy(start_block(S.shape[0], b, i)).cuda() for i, (S, *_rest) in enumerate(members)]
        wide = [torch.cat([x, x], 1)[:, :b] for x in xs]  # rows further apart than b
        cols = [x.t().contiguous() for x in xs]
        outs = [torch.zeros_like(c) for c in cols]
        xp, yp = ((C.c_void_p * len(xs))(*[t.data_ptr() for t in ts]) for ts in (cols, outs))
        torch.cuda.synchronize()
        assert kf.lib().kf_batch_apply_filter(bt._h, C.cast(xp, C.c_void_p), C.cast(yp, C.c_void_p), b) == 0
        for y, w, o in zip(bt.apply_filter(xs), bt.apply_filter(wide), outs):
            assert torch.equal(y, o.t()) and torch.equal(w, y)
