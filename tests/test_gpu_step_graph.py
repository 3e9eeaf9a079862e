"""Filter applications whose middle steps are replayed from a recording
against launches of every step (the allocation-free entry point, which records
nothing), bit for bit: the same kernels on the same buffers."""

import numpy as np
import pytest

from synth import start_block
from synth.grids import grid_problem, jittered_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stream", ["default", "own"])
@pytest.mark.parametrize("stepper", [2, 4])
@pytest.mark.parametrize(
    "kind,b,precision",
    # beyond several steps per launch: a value per offset and per row, widths
    # that need the load launch, both precisions
    [("cube44", 1, "fp64"), ("cube44", 3, "mixed"), ("cube41", 4, "fp64"), ("jitter26", 2, "fp64"),
     ("jitter26", 8, "mixed")],
)
def test_replayed_steps_bitwise(kind, b, precision, stepper, stream):
    import torch

    from paper_2402_08515_amd import kf

    print(f"case step graph {kind} b={b} {precision} stepper={stepper} {stream}", flush=True)
    n = int(kind[-2:])
    S, m = jittered_problem(3, n, 0.2, 3) if kind.startswith("jitter") else grid_problem(3, n)[:2]
    tau = 1.8 / np.sqrt(np.abs(S).sum(1).max() / m.min())
    s = torch.cuda.default_stream() if stream == "default" else torch.cuda.Stream()
    with torch.cuda.stream(s):
        for L in (11, 12, 30):  # too few steps to record, the fewest, more
            P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, L, precision=precision, stepper=stepper)
            y = torch.empty((S.shape[0], b), dtype=torch.float64, device="cuda")
            for rep in range(15):  # launched, recorded (the sixth), replayed; then again after new weights
                if rep == 7:
                    P.set_weights(np.linspace(1.0, 0.1, L))
                x = torch.from_numpy(start_block(S.shape[0], b, rep)).cuda()
                got = P.apply_filter(x)
                P.apply_filter_noalloc(x, y)
                assert torch.equal(got, y), (L, rep, (got - y).abs().max())
            # another width in between, and the first again
            x1 = torch.from_numpy(start_block(S.shape[0], 1, 7)).cuda()
            y1 = torch.empty_like(x1)
            for _ in range(7):
                P.apply_filter_noalloc(x1, y1)
                assert torch.equal(P.apply_filter(x1), y1), L
            P.apply_filter_noalloc(x, y)
            for _ in range(7):
                assert torch.equal(P.apply_filter(x), y), L
        torch.cuda.synchronize()


def test_applications_under_the_callers_capture():
    """A problem that replays its steps still can be captured by its caller:
    the recording then holds plain launches."""
    import torch

    from paper_2402_08515_amd import kf

    print("case step graph under capture", flush=True)
    S, m = grid_problem(3, 44)[:2]
    tau = 1.8 / np.sqrt(np.abs(S).sum(1).max() / m.min())
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, 30)
        x = torch.from_numpy(start_block(S.shape[0], 1, 1)).cuda()
        want = [P.apply_filter(x) for _ in range(7)][-1]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            y = P.apply_filter(x)
        for _ in range(3):
            y.zero_()
            g.replay()
            assert torch.equal(y, want)
            assert torch.equal(P.apply_filter(x), want)
        torch.cuda.synchronize()
