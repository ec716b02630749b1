"""Jacobi kernel at the sizes and scales where its slot layout can go wrong:
one pair, odd sizes (dummy row), the last sizes that change its split over the
wavefronts, equal diagonals (the rotation's sign tie), zero couplings and
matrices far from unit scale."""
import numpy as np
import pytest

import paper_2201_07498_amd as lz

pytestmark = pytest.mark.gpu


def _check(alpha, beta):
    m = alpha.size
    theta, S, sweeps = lz.tridiag_eig(alpha, beta)
    T = np.diag(alpha) + (np.diag(beta, 1) + np.diag(beta, -1) if m > 1 else 0.0)
    norm = np.linalg.norm(T) or 1.0
    # Backward error of cyclic Jacobi: each of the sweeps applies m - 1 rounds
    # of rotations that are each exact to a few units of the last place.
    tol = 8.0 * max(1, sweeps) * m * 2.0 ** -53
    assert 1 <= sweeps <= 15
    assert np.max(np.abs(np.sort(theta) - np.linalg.eigvalsh(T))) <= tol * norm
    assert np.max(np.abs(S.T @ S - np.eye(m))) <= tol
    assert np.max(np.abs((T / norm) @ S - S * (theta / norm))) <= tol


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 11, 12, 23, 24, 33, 47, 48, 49, 62, 63, 64])
@pytest.mark.parametrize("kind", ["random", "equal_diagonal", "zero_couplings", "tiny", "huge"])
def test_jacobi_layout_edges(m, kind):
    rng = np.random.default_rng(100 * m + len(kind))
    alpha, beta = rng.normal(size=m), rng.normal(size=max(m - 1, 0))
    if kind == "equal_diagonal":
        alpha[:] = 0.5
        beta[:] = 1.0
    if kind == "zero_couplings":
        beta[::3] = 0.0
        alpha[::4] = 0.0
    scale = {"tiny": 2.0 ** -700, "huge": 2.0 ** 700}.get(kind, 1.0)
    theta, S, _ = lz.tridiag_eig(alpha, beta)
    _check(alpha, beta)
    if scale != 1.0:                    # a power of two only moves the exponents
        theta2, S2, _ = lz.tridiag_eig(alpha * scale, beta * scale)
        assert np.array_equal(theta2, theta * scale)
        assert np.array_equal(S2, S)


def test_jacobi_zero_matrix():
    theta, S, sweeps = lz.tridiag_eig(np.zeros(7), np.zeros(6))
    assert sweeps == 1 and not theta.any() and np.array_equal(S, np.eye(7))
