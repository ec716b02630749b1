"""Report and output kernels at the edges of their tiles: 32-row steps and
16-column blocks of the Gram kernel (also with padding between the columns),
and solves whose K is around a column block or whose rows are around a
wavefront's 64, against the same quantities of the returned vectors."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import device_csr, device_values

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("n,c", [(1, 2), (31, 15), (32, 16), (33, 17), (65, 32), (127, 33), (129, 48), (4097, 49),
                                 (200_001, 64)])
def test_gram_tiles_with_padded_columns(n, c, precision):
    rng = np.random.default_rng(7 * n + c)
    X = synth.round_values(rng.standard_normal((n, c)) / np.sqrt(n), precision).reshape(n, c)
    pad = 3                                   # odd distance: columns start at any multiple of the element
    flat = np.full((c, n + pad), np.nan)      # what lies between the columns must not be read into the sums
    flat[:, :n] = X.T
    dX = device_values(flat.ravel(), precision).view(c, n + pad).T[:n]
    want = np.max(np.abs(X.T @ X - np.eye(c)))
    # Two sums of n products each, in any order: n units of the last place of
    # the sum of moduli, at most the largest column norm squared.
    tol = 2.0 * n * EPS * max(1.0, float(np.max(np.sum(X * X, axis=0))))
    assert abs(lz.ortho_loss(dX, precision) - want) <= tol


@pytest.mark.parametrize("reorder", ["off", "hubs"])
@pytest.mark.parametrize("n,K,m", [(65, 1, 5), (130, 15, 40), (200, 16, 40), (257, 17, 50), (300, 32, 60), (300, 33, 64),
                                   (511, 48, 64), (1000, 49, 64), (1029, 64, 64)])
def test_vectors_and_metrics_around_column_blocks(n, K, m, reorder):
    rp, c, v = synth.er(n, 8.0, seed=n + K)
    drp, dc, dv = device_csr(rp, c, v, "fp64")
    vals, vecs, rep = lz.topk(drp, dc, dv, K, m, "fp64", seed=3, reorder=reorder)
    torch.cuda.synchronize()
    vals, Y = vals.cpu().numpy(), vecs.cpu().numpy()
    Y = Y if Y.shape == (n, K) else Y.T
    # A column's norm and its Gram entries: sums of n products of unit vectors.
    tol = 4.0 * n * EPS
    assert np.max(np.abs(np.sum(Y * Y, axis=0) - 1.0)) <= tol
    top = np.argmax(np.abs(Y), axis=0)
    assert np.all(Y[top, np.arange(K)] > 0.0)
    assert abs(rep["ritz_ortho_loss"] - oracle.ortho_loss(Y)) <= tol
    # acos has slope up to 1 away from parallel vectors; the Gram entries of a
    # report that holds are far from 1.
    if rep["ritz_ortho_loss"] < 0.5:
        assert abs(rep["mean_angle_deg"] - oracle.mean_angle_deg(Y)) <= 2.0 * tol * 180.0 / np.pi + 180.0 * 4 * EPS
    # Residual vectors: products of rows of A, then n squares; both sides round
    # relative to |A| |y|, not to the difference.
    norm = max(1.0, float(np.max(np.abs(vals))))
    ab, _ = oracle.residuals(rp, c, v, vals, Y)
    row = float(np.max(np.diff(rp)))
    absA = float(np.max(np.bincount(np.repeat(np.arange(n), np.diff(rp)), weights=np.abs(v), minlength=n)))
    assert np.max(np.abs(rep["abs_resid"] - ab)) <= (n + row) * EPS * 4.0 * max(norm, absA)
