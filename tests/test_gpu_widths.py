"""Block widths that alternate on one problem: the step buffers stay where they
are, so a recording the caller made of one width survives applications of the
others, and the results are those of a problem of each width's own."""

import numpy as np
import pytest

from synth import start_block
from synth.grids import grid_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stepper", [2, 4])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_recorded_width_survives_the_others(precision, stepper):
    import torch

    from paper_2402_08515_amd import kf

    print(f"case widths {precision} stepper={stepper}", flush=True)
    # (300 cells: several steps per launch for one and four vectors, not for eight)
    S, m, _ = grid_problem(2, 300)
    tau = 1.8 / np.sqrt(8.0 * 300 * 300)
    make = lambda: kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, 40, precision=precision, stepper=stepper)  # noqa: E731
    x = {b: torch.from_numpy(start_block(S.shape[0], b, b)).cuda() for b in (1, 3, 8, 16)}
    want = {b: make().apply_filter(x[b]) for b in x}
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        P = make()
        for b in (8, 1, 16, 3):
            assert torch.equal(P.apply_filter(x[b]), want[b]), b
        torch.cuda.synchronize()
        graphs, ys = {}, {}
        for b in (1, 16):
            graphs[b] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graphs[b], stream=s):
                ys[b] = P.apply_filter(x[b])
        for rep in range(3):
            for b in (16, 1):
                ys[b].zero_()
                graphs[b].replay()
                assert torch.equal(ys[b], want[b]), (rep, b)
            for b in (8, 1, 3, 16):
                assert torch.equal(P.apply_filter(x[b]), want[b]), (rep, b)
        torch.cuda.synchronize()
