"""The eigensolver on matrices far from norm one.  Scaling by a power of two
is exact, so eigenvalues scale with it; the tolerances are those of the same
matrices at norm one (a few roundings of the bisection)."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _second_difference(k):
    return 2.0 * np.eye(k) - np.diag(np.ones(k - 1), 1) - np.diag(np.ones(k - 1), -1)


# (2^-514: the power of two that brings the matrix to norm one has an infinite
# square; off-diagonals are powers of two, so that their squares are exact
# although subnormal)
@pytest.mark.parametrize("exponent", [-536, -520, -514, -513, -512, -500, -100, 0, 100, 500])
@pytest.mark.parametrize("k", [20, 50, 300])
def test_eigenvalues_scale_with_the_matrix(k, exponent):
    from paper_2402_08515_amd import kf

    print(f"case sym_eig scale 2^{exponent} k={k}", flush=True)
    T, s = _second_difference(k), 2.0**exponent
    theta = kf.sym_eig(T * s) / s
    np.testing.assert_allclose(theta, np.linalg.eigvalsh(T), atol=1e-13)


@pytest.mark.parametrize("exponent", [-900, -600, -530, 530, 600, 900])
@pytest.mark.parametrize("k", [20, 50, 300])
def test_diagonal_matrices_of_any_scale(k, exponent):
    from paper_2402_08515_amd import kf

    print(f"case sym_eig diagonal scale 2^{exponent} k={k}", flush=True)
    d = np.sort(np.random.default_rng(k).uniform(1.0, 2.0, size=k))
    np.testing.assert_allclose(kf.sym_eig(np.diag(d[::-1]) * 2.0**exponent), d * 2.0**exponent, rtol=1e-14)


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("k", [50, 300])
def test_repeated_diagonal_entries_at_a_section_point(k, fused):
    """The bisection's first points depend on the extreme entries alone: runs
    of diagonal entries equal to some of them (rounded as a product and a sum,
    or once) give it pivots of zero row after row."""
    from fractions import Fraction

    from paper_2402_08515_amd import kf

    print(f"case sym_eig section points k={k} fused={fused}", flush=True)
    d = np.linspace(1.0, 2.0, k)
    widen = 2.0 * np.finfo(float).eps * 2.0
    lo, hi = 1.0 - widen - np.finfo(float).tiny, 2.0 + widen + np.finfo(float).tiny
    h = (hi - lo) / 65.0
    for i, point in enumerate((20, 41)):
        x = float(Fraction(lo) + point * Fraction(h)) if fused else lo + point * h
        d[8 + 16 * i : 24 + 16 * i] = x
    np.testing.assert_allclose(kf.sym_eig(np.diag(d)), np.sort(d), rtol=1e-14)


@pytest.mark.parametrize("exponent", [-500, -480, -400, 0, 400, 500])
@pytest.mark.parametrize("k", [20, 50, 300])
def test_eigenvectors_scale_with_the_matrix(k, exponent):
    """Vectors of a part of the spectrum: unit norm, orthogonal, and
    eigenvectors of the matrix brought back to norm one (tolerances of the
    eigensolver's other tests)."""
    from paper_2402_08515_amd import kf

    print(f"case sym_eig vectors scale 2^{exponent} k={k}", flush=True)
    T, s = _second_difference(k), 2.0**exponent
    theta, Y = kf.sym_eig(T * s, 1.0 * s, 3.0 * s, vectors=True)
    sel = theta[(theta >= 1.0 * s) & (theta <= 3.0 * s)] / s
    assert Y.shape == (k, sel.size) and sel.size >= k // 4
    assert np.abs(T @ Y - Y * sel).max() <= 1e-11 * 4.0
    assert np.abs(Y.T @ Y - np.eye(sel.size)).max() <= 1e-10


@pytest.mark.parametrize("exponent", [-900, -600, 600, 900])
@pytest.mark.parametrize("k", [20, 50, 300])
def test_eigenvectors_of_diagonal_matrices_of_any_scale(k, exponent):
    from paper_2402_08515_amd import kf

    print(f"case sym_eig diagonal vectors scale 2^{exponent} k={k}", flush=True)
    d, s = np.linspace(1.0, 2.0, k), 2.0**exponent
    theta, Y = kf.sym_eig(np.diag(d) * s, 1.2 * s, 1.8 * s, vectors=True)
    sel = theta[(theta >= 1.2 * s) & (theta <= 1.8 * s)] / s
    assert Y.shape == (k, sel.size) and sel.size >= k // 2
    assert np.abs(d[:, None] * Y - Y * sel).max() <= 1e-11 * 2.0
    assert np.abs(Y.T @ Y - np.eye(sel.size)).max() <= 1e-10


@pytest.mark.parametrize("off", [1e-100, 1e-160, 1e-200, 1e-290])
@pytest.mark.parametrize("k", [3, 20, 50, 300])
def test_eigenvectors_beside_tiny_off_diagonals(k, off):
    """Where a shift equals a diagonal entry, the off-diagonal below it is the
    pivot and its inverse the largest entry of the iterate, however tiny."""
    from paper_2402_08515_amd import kf

    print(f"case sym_eig off-diagonal {off} k={k}", flush=True)
    d = np.random.default_rng(k).standard_normal(k)
    A = np.diag(d) + np.diag(np.full(k - 1, off), 1) + np.diag(np.full(k - 1, off), -1)
    theta, Y = kf.sym_eig(A, -10.0, 10.0, vectors=True)
    np.testing.assert_allclose(theta, np.sort(d), atol=1e-14)
    assert Y.shape == (k, k)
    assert np.abs(A @ Y - Y * theta).max() <= 1e-11 * np.abs(d).max()
    assert np.abs(Y.T @ Y - np.eye(k)).max() <= 1e-10
