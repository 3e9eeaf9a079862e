"""The network's kernels at the sizes where their tiling can go wrong (one
staged group of 64 rows, an odd number of groups, many) against the FP64
reference with bfloat16 operands, and the in-place Adam step against the
gradient it is made from."""

import numpy as np
import pytest

from oracle import mlp
from synth.workloads import filter_samples

pytestmark = pytest.mark.gpu


def _theta(seed):
    rng = np.random.default_rng(seed)
    t = mlp.init_params(seed)
    t[-(128 * 512 + 512):] = 0.3 * rng.standard_normal(128 * 512 + 512)
    return t.astype(np.float32)


@pytest.mark.parametrize("rows", [64, 192, 1024])
def test_gradient_at_tile_edges(rows):
    """As in the element-by-element gradient test: entries within 1e-3 of
    their layer's largest, the loss within 1e-5."""
    from paper_2402_08515_amd import kf

    print(f"case gradient rows={rows}", flush=True)
    theta, s = _theta(rows), filter_samples(rows, stream=0)
    loss, g = kf.Mlp(theta).loss_grad(s)
    ref_loss, ref = mlp.loss_and_grad(theta.astype(np.float64), s, bf16=True)
    assert loss == pytest.approx(ref_loss, rel=1e-5)
    off = 0
    for shape in mlp.SHAPES:
        k = int(np.prod(shape))
        a, b = g[off:off + k].astype(np.float64), ref[off:off + k]
        assert np.abs(a - b).max() <= 1e-3 * np.abs(b).max(), shape
        off += k


@pytest.mark.parametrize("batch,rows", [(64, 64), (192, 200)])
def test_adam_step_follows_the_gradient(batch, rows):
    """One training step against Adam's formula on the gradient of the same
    rows.  The step is lr times a ratio of magnitude one in float32 (a dozen
    roundings, 1e-6 of it) and a parameter is rounded once; ratios of tiny
    gradients lose relative accuracy through eps, which the same formula in
    float64 on the float32 gradient shares.  Afterwards the network must equal
    a new one made from its parameters, bit for bit (the weights are kept in
    three layouts)."""
    from paper_2402_08515_amd import kf

    print(f"case adam batch={batch} rows={rows}", flush=True)
    theta, s = _theta(7), filter_samples(rows, stream=0)
    order = np.random.default_rng(1).permutation(rows).astype(np.int32)
    _, g = kf.Mlp(theta).loss_grad(s[order[:batch]])
    net = kf.Mlp(theta)
    lr = 1e-3
    hist = net.train(s, order, 1, batch, lr)
    p = net.params()
    g64 = g.astype(np.float64)
    m1, m2 = 0.1 * g64, 0.001 * g64**2
    step = lr * (m1 / 0.1) / (np.sqrt(m2 / 0.001) + 1e-8)
    # 1 - 0.9 and 1 - 0.999 are float32 differences on one side of each ratio
    assert np.abs(p - (theta - step)).max() <= lr * 1e-4 + 1.2e-7 * np.abs(theta).max()
    loss, _ = kf.Mlp(theta).loss_grad(s[order[:batch]], want_grad=False)
    assert hist[0] == pytest.approx(loss, rel=1e-6)
    la, ga = net.loss_grad(s[order[:64]])
    lb, gb = kf.Mlp(p).loss_grad(s[order[:64]])
    assert la == lb and np.array_equal(ga, gb)
