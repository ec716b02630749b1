"""Relabelling with the table of hot labels (2^22 rows and more): columns in
the table, columns that lost their slot and columns past the hot ones, plain and
in sweep blocks, against the solve that is not relabelled."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import scipy.sparse as sp  # noqa: E402

import paper_2201_07498_amd as lz  # noqa: E402
from gpu_util import device_csr  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(1 << 22) - 1, 1 << 22, (1 << 22) + 12345])
def matrix(request):
    n = request.param
    rng = np.random.default_rng(n)
    hubs = rng.choice(n, 400_000, replace=False)          # more than the table takes
    pick = (400_000 * rng.random(3_000_000) ** 4).astype(np.int64)
    r = np.concatenate([np.arange(n - 1), hubs[pick]])
    c = np.concatenate([np.arange(1, n), rng.integers(0, n, pick.size)])
    v = rng.uniform(0.1, 1.0, r.size)
    a = sp.coo_matrix((v, (r, c)), shape=(n, n))
    a = (a + a.T).tocsr()
    a.sum_duplicates()
    return a.indptr.astype(np.int64), a.indices.astype(np.int32), a.data


@pytest.mark.parametrize("sweep", ["off", "on"])
def test_relabelled_solve_matches_the_plain_one(matrix, sweep):
    rp, c, v = matrix
    n, K, m = rp.size - 1, 2, 5
    csr = device_csr(rp, c, v, "fp64")
    _, _, plain = lz.topk(*csr, K, m, "fp64", seed=3, reorder="off", sweep="off")
    vals, vecs, rep = lz.topk(*csr, K, m, "fp64", seed=3, reorder="hubs", sweep=sweep)
    assert rep["reordered"]
    # Sums over n rows and at most a few thousand entries a row in another
    # order, m steps of them.
    tol = m * 2.0 * n * 2.0 ** -53 * np.max(np.abs(plain["theta"]))
    assert np.max(np.abs(rep["alpha"] - plain["alpha"])) <= tol
    assert np.max(np.abs(rep["beta"] - plain["beta"])) <= tol
    # Each pair's residual, with A as the caller gave it.
    a = sp.csr_matrix((v, c, rp), shape=(n, n))
    y = vecs.cpu().numpy() if vecs.shape == (n, K) else vecs.cpu().numpy().T
    th = vals.cpu().numpy()
    ab = np.linalg.norm(a @ y - y * th, axis=0)
    assert np.max(np.abs(ab - rep["abs_resid"])) <= tol
