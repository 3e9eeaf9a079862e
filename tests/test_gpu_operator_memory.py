"""An operator stepped as stencils takes no more device memory than the same
operator in its stored entries (index_bytes fixed)."""

import numpy as np
import pytest

from synth.grids import grid_problem, jittered_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", ["grid", "jitter"])  # one value per offset; a value per row
def test_one_form_of_an_operator_is_kept(kind, precision):
    import torch

    from paper_2402_08515_amd import kf

    S, m = (grid_problem(3, 64)[:2]) if kind == "grid" else jittered_problem(3, 48, 0.2, 3)
    tau = 1.8 / np.sqrt((np.abs(S).sum(1).A1 / m).max())

    def used(index_bytes):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        P = kf.Problem(S, m, 0.3 / tau, 0.5 / tau, tau, 20, precision=precision, index_bytes=index_bytes)
        torch.cuda.synchronize()
        took = before - torch.cuda.mem_get_info()[0]
        P.close()
        return took

    used(2)  # (what the runtime allocates once)
    stored, stencil = used(2), used(0)
    print(f"case operator memory {kind} {precision}: stored entries {stored}, stencils {stencil}", flush=True)
    assert 0 < stencil <= stored
