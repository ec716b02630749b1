"""Which solves lay out the tail columns of the sweep blocks ahead, and the forms
that no smaller test reaches: captured in a graph, positions past 4 GiB of
gathered entries, and 16-bit columns past the last panel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402
import synth  # noqa: E402
from gpu_util import device_csr  # noqa: E402

pytestmark = pytest.mark.gpu

SIZE = {"fp64": 8, "fp32": 4, "bf16": 2}
DTYPE = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}
HEAD, PANEL, PANELS_MAX = 4 << 20, 128 << 10, 512       # bytes of x, bytes, count
KW = dict(reorder="hubs", sweep="on")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_panels_by_size(precision):
    # The sizes at which the split of x changes, with the entries per row that the
    # tests of the tail columns have (1.5 and 0.5 beside the diagonal).
    head, panel = HEAD // SIZE[precision], PANEL // SIZE[precision]
    for rows, per_row, want in ((head - 5, 2.5, 0), (head, 2.5, 0), (head + 1, 2.5, 1), (head + panel, 2.5, 1),
                                (head + panel + 1, 2.5, 2), (head + 5 * panel // 2 + 77, 2.5, 3),
                                (head + PANELS_MAX * panel, 1.5, PANELS_MAX),
                                (head + PANELS_MAX * panel + 40_001, 1.5, PANELS_MAX)):
        assert lz.sweep_panels(rows, int(per_row * rows), 2, 5, precision, **KW) == want, (rows, want)
    assert lz.sweep_panels(head + panel, 3 * head, 2, 5, precision, sweep="off") == 0
    assert lz.sweep_panels(head + panel, 3 * head, 2, 5, precision, sweep="on", reorder="off") == 0


def test_tail_columns_in_hip_graph_replay_bitwise():
    rp, c, v = synth.rmat_n(1_300_003, 4.0, seed=5)
    n, K, m = rp.size - 1, 3, 8
    drp, dc, dv = device_csr(rp, c, v, "fp32")
    assert lz.sweep_panels(n, c.size, K, m, "fp32", **KW) > 1
    ws = torch.empty(lz.workspace_size(n, c.size, K, m, "fp32", **KW), dtype=torch.uint8, device="cuda:0")
    out = (torch.empty(K, dtype=torch.float64, device="cuda:0"),
           torch.empty(K, n, dtype=torch.float64, device="cuda:0"))
    d_rep = torch.empty(lz.REPORT_BYTES, dtype=torch.uint8, device="cuda:0")
    vals, vecs, rep = lz.topk(drp, dc, dv, K, m, "fp32", seed=11, workspace=ws, **KW)
    assert rep["spmv_layout"] == 4
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            lz.topk_async(drp, dc, dv, K, m, "fp32", seed=11, workspace=ws, out=out, d_report=d_rep, stream=side, **KW)
    torch.cuda.current_stream().wait_stream(side)
    other = device_csr(*synth.er(3000, 9.0, seed=6), "fp64")
    for replay in range(3):
        for t in (*out, d_rep):
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = lz.report_from_device(d_rep, K, m)
        assert got["status"] == 0 and np.array_equal(got["alpha"], rep["alpha"]), replay
        assert torch.equal(out[0], vals) and torch.equal(out[1].T, vecs), replay
        lz.topk(*other, 4, 12, "fp64", seed=replay)      # eager work between replays
        torch.cuda.synchronize()


def circulant(n, pairs, precision):
    """Symmetric circulant CSR matrix on the GPU: the diagonal and `pairs` offsets
    each way, spread over the whole row, with weights exact in every precision."""
    rng = np.random.default_rng(pairs)
    offs = np.unique(rng.integers(1, n // 2, 4 * pairs))
    offs = rng.choice(offs, pairs, replace=False)
    offs = [0] + [int(s * o) for o in offs for s in (1, -1)]
    w = [2.0] + [float(x) for x in rng.choice([0.25, 0.5, 0.75, 1.0], pairs) for _ in range(2)]
    row = torch.arange(n, dtype=torch.int64, device="cuda:0")
    col = torch.empty((n, len(offs)), dtype=torch.int32, device="cuda:0")
    for k, o in enumerate(offs):
        col[:, k] = (row + o) % n
    val = torch.tensor(w, device="cuda:0").to(DTYPE[precision]).repeat(n)
    rp = torch.arange(n + 1, dtype=torch.int64, device="cuda:0") * len(offs)
    return rp, col.reshape(-1), val


@pytest.mark.parametrize("precision,n,pairs,tol", [
    ("fp64", (1 << 22) + 4321, 64, 1e-12),               # xg past 4 GiB
    ("bf16", 37_800_001, 29, 1e-3),                      # xg past 4 GiB, columns past the last panel
])
def test_wide_positions_and_columns_past_the_last_panel(precision, n, pairs, tol):
    K, m = 2, 4
    print(f"sweep tail {precision} n={n} pairs={pairs}", flush=True)
    csr = circulant(n, pairs, precision)
    nnz = csr[1].numel()
    assert nnz * SIZE[precision] > 1 << 32 and nnz < (1 << 32) - 1
    panels = lz.sweep_panels(n, nnz, K, m, precision, **KW)
    assert panels == min(PANELS_MAX, -(-(n * SIZE[precision] - HEAD) // PANEL))
    reps = []
    for sweep in ("off", "on"):
        vals, vecs, rep = lz.topk(*csr, K, m, precision, seed=3, reorder="hubs", sweep=sweep)
        reps.append((vals.cpu().numpy(), rep))
        del vecs
        lz.release_memory()
    (a, ra), (b, rb) = reps
    assert rb["spmv_layout"] == 4 and ra["restarts"] == rb["restarts"] == 0
    # Two summation orders of the same SpMV over a short run: rounding of the
    # stored vectors, as in the tests at smaller sizes.
    tol *= np.max(np.abs(ra["theta"]))
    for x, y in ((a, b), (ra["alpha"], rb["alpha"]), (ra["beta"], rb["beta"])):
        assert np.max(np.abs(x - y)) <= tol
    # The recurrence of the sweep solve against the matrix: with A V = V T + beta v e^T
    # the residual of pair k, which the report takes from the tiles in FP64, is
    # beta |s_mk|, up to the rounding u of the stored columns (||A|| is the row sum
    # of a circulant).  A gather from a wrong place leaves a residual of the size of
    # the matrix' bulk, several times the bound.
    top = float(csr[2][: nnz // n].double().sum())
    lam, S = np.linalg.eigh(np.diag(rb["alpha"]) + np.diag(rb["beta"][1:m], 1) + np.diag(rb["beta"][1:m], -1))
    pick = np.argsort(-np.abs(lam))[:K]
    u = {"fp64": np.sqrt(n) * 2.0 ** -53, "bf16": 2.0 ** -9}[precision]
    want = rb["beta_last"] * np.abs(S[m - 1, pick])
    print(f"residuals {rb['abs_resid']}, recurrence {want}", flush=True)
    assert np.max(np.abs(rb["abs_resid"] - want)) <= 4.0 * np.sqrt(m) * top * u
    del csr
    torch.cuda.empty_cache()
