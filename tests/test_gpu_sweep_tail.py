"""Sweep blocks with tail columns (x longer than its directly gathered head):
the sizes where the split of x into head, LDS panels and the part past the last
panel changes, against the same solve on row-ordered tiles."""
import numpy as np
import pytest
import torch

import paper_2201_07498_amd as lz
import synth
from gpu_util import device_csr

pytestmark = pytest.mark.gpu

SIZE = {"fp64": 8, "fp32": 4, "bf16": 2}
HEAD, PANEL, PANELS_MAX = 4 << 20, 128 << 10, 512       # bytes of x, bytes, count
# Ritz values of a short run on two summation orders of the same SpMV: rounding
# of the stored vectors (BF16 flips whole units of 2^-8 of single entries).
TOL = {"fp64": 1e-12, "fp32": 1e-6, "bf16": 1e-3}


def _both(rp, c, v, precision, K, m):
    csr = device_csr(rp, c, synth.round_values(v, precision), precision)
    out = []
    for sweep in ("off", "on"):
        vals, vecs, rep = lz.topk(*csr, K, m, precision, seed=3, reorder="hubs", sweep=sweep)
        out.append((vals.cpu().numpy(), rep))
    (a, ra), (b, rb) = out
    assert rb["spmv_layout"] & 15 == 4
    assert ra["restarts"] == rb["restarts"] == 0
    tol = TOL[precision] * np.max(np.abs(ra["theta"]))
    assert np.max(np.abs(ra["alpha"] - rb["alpha"])) <= tol
    assert np.max(np.abs(ra["beta"] - rb["beta"])) <= tol
    assert np.max(np.abs(a - b)) <= tol


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("extra", ["one_column", "panel", "panel_and_one", "ragged"])
def test_tail_columns_match_tiles(precision, extra):
    head, panel = HEAD // SIZE[precision], PANEL // SIZE[precision]
    n = head + {"one_column": 1, "panel": panel, "panel_and_one": panel + 1, "ragged": 5 * panel // 2 + 77}[extra]
    # Every column is gathered: a sparse uniform graph with a full diagonal.
    _both(*synth.er(n, 1.5, seed=5), precision, 2, 5)


def test_columns_past_the_last_panel_match_tiles():
    n = (HEAD + PANELS_MAX * PANEL) // 8 + 40_001
    print(f"sweep tail fp64 n={n}", flush=True)
    _both(*synth.er(n, 0.5, seed=6), "fp64", 2, 3)


def test_tail_columns_on_power_law_rows_match_tiles():
    _both(*synth.rmat_n(700_001, 9.0, seed=7), "fp64", 4, 12)
