"""The eigensolver at the orders where its reduction changes hands: the last
128 reflectors move into one workgroup, registers hold 4, 8 or 16 rows per
lane, larger orders keep their vectors in LDS first.  Spectrum fixed by
construction; tolerances of the eigensolver's other tests (rounding of the
reduction, about sqrt(k) ulps of the largest eigenvalue)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [63, 64, 65, 127, 128, 129, 130, 255, 256, 257, 384, 512, 513, 769, 1025])
def test_eigenpairs_at_the_edges(k):
    from paper_2402_08515_amd import kf

    print(f"case sym_eig edge k={k}", flush=True)
    rng = np.random.default_rng(900 + k)
    lam = np.sort(rng.uniform(-3.0, 5.0, size=k))
    Q, _ = np.linalg.qr(rng.standard_normal((k, k)))
    A = (Q * lam) @ Q.T
    lo, hi = lam[k // 3] - 1e-9, lam[k // 3 + 20] + 1e-9
    theta, Y = kf.sym_eig(A, lo, hi, vectors=True)
    assert np.abs(theta - lam).max() <= 1e-12 * 5.0 * max(1.0, np.sqrt(k) / 8)
    sel = theta[(theta >= lo) & (theta <= hi)]
    assert Y.shape == (k, sel.size) and sel.size >= 20
    assert np.abs(A @ Y - Y * sel).max() <= 1e-11 * 5.0
    assert np.abs(Y.T @ Y - np.eye(sel.size)).max() <= 1e-10


@pytest.mark.parametrize("k", [50, 200, 300])
def test_split_and_constant_matrices(k):
    """Zero off-diagonals (diagonal matrices, blocks), equal diagonals and a
    zero matrix: the counts meet zero pivots and the reflectors are trivial."""
    from paper_2402_08515_amd import kf

    rng = np.random.default_rng(k)
    d = np.sort(rng.uniform(1.0, 2.0, size=k))
    np.testing.assert_allclose(kf.sym_eig(np.diag(d[::-1].copy())), d, rtol=1e-14)
    np.testing.assert_allclose(kf.sym_eig(3.0 * np.eye(k)), np.full(k, 3.0), rtol=1e-14)
    assert np.abs(kf.sym_eig(np.zeros((k, k)))).max() <= 1e-300
    T = 2.0 * np.eye(k) - np.diag(np.ones(k - 1), 1) - np.diag(np.ones(k - 1), -1)
    T[k // 2, k // 2 - 1] = T[k // 2 - 1, k // 2] = 0.0
    np.testing.assert_allclose(kf.sym_eig(T), np.linalg.eigvalsh(T), atol=1e-13)
