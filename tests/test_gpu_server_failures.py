"""A request that fails on the device leaves the caller's buffers untouched, also
where its arena block held an earlier request's results."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402
import synth  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_graphs", [False, True])
@pytest.mark.parametrize("fault,status", [("column", -1), ("nan", -7)])
def test_failed_request_leaves_its_buffers_untouched(fault, status, use_graphs):
    rp, c, v = synth.er(3000, 9.0, seed=1)
    bad_c, bad_v = c.copy(), v.copy()
    if fault == "column":
        bad_c[17] = 3000                      # outside [0, n): refused by the device's input checks
    else:
        bad_v[17] = np.nan
    with lz.Server(1 << 26, max_slots=1, use_graphs=use_graphs) as srv:
        for _ in range(2):
            good = srv.submit(rp, c, v, 4, 16, "fp64", want_vectors=True)
            vals, vecs, res = srv.wait(good)
            assert res["status"] == 0 and np.all(vals != 0.0)
            assert np.allclose(np.linalg.norm(vecs, axis=0), 1.0, atol=1e-12)
            bad = srv.submit(rp, bad_c, bad_v, 4, 16, "fp64", want_vectors=True)
            vals, vecs, res = srv.wait(bad)
            assert res["status"] == status
            # The buffers of Server.submit start as zeros.
            assert not vals.any() and not vecs.any() and not res["resid"].any()
