"""Tridiagonal matrices with NaN or infinite entries: which ones the Jacobi solve
returns and which it refuses, with and without the dummy row of an odd size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402

pytestmark = pytest.mark.gpu
NAN, INF = np.nan, np.inf


@pytest.mark.parametrize("diag", [[NAN], [INF], [-INF], [0.0], [5e-324], [INF, 1.0], [INF, 1.0, -2.0], [3.0, INF, -INF]])
def test_decoupled_diagonals_come_back(diag):
    # No pair has anything to rotate (an infinite norm makes every coupling negligible).
    theta, S, sweeps = lz.tridiag_eig(np.array(diag), np.zeros(len(diag) - 1))
    assert np.array_equal(theta, diag, equal_nan=True) and sweeps == 1
    assert np.array_equal(S, np.eye(len(diag)))


@pytest.mark.parametrize("diag,off", [([1.0, NAN], [0.0]), ([NAN, 1.0, 2.0], [0.0, 0.0]), ([1.0, 2.0], [NAN]),
                                      ([1.0, 2.0, 3.0], [0.5, NAN])])
def test_nan_is_refused(diag, off):
    with pytest.raises(lz.LanczosError) as e:
        lz.tridiag_eig(np.array(diag), np.array(off))
    assert e.value.code == -6
