"""The stored oracle solves that bench.py measures its errors against belong to
the matrices that it builds (runs without a GPU)."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("workload,stored", [("rmat20", False), ("rmat23", True), ("rmat26", True), ("er10k", False)])
def test_reference_of_a_workload(bench, workload, stored):
    # (The stored R-MAT 20 solve is of BF16-rounded values, which the benchmark does not round.)
    assert (bench.golden(workload) is not None) == stored
