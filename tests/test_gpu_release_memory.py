"""Device memory that the library keeps between calls is bounded and can be given back."""
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402
import synth  # noqa: E402
from gpu_util import device_csr  # noqa: E402

pytestmark = pytest.mark.gpu


def test_release_memory():
    csr = device_csr(*synth.er(200_000, 9.0, seed=3), "fp64")
    out = (torch.empty(8, dtype=torch.float64, device="cuda:0"),
           torch.empty(8, 200_000, dtype=torch.float64, device="cuda:0"))

    def solve():
        lz.topk(*csr, 8, 24, "fp64", seed=1, out=out)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    solve()                                   # code objects, streams and scratch of the first call
    lz.release_memory()
    before = torch.cuda.mem_get_info()[0]
    kept = before - solve()
    vals = out[0].clone()
    need = lz.workspace_size(200_000, csr[1].numel(), 8, 24, "fp64")
    print(f"workspace {need} bytes, kept {kept}", flush=True)
    assert 0 < kept <= 2 << 30
    lz.release_memory()
    assert torch.cuda.mem_get_info()[0] == before
    solve()
    assert torch.equal(out[0], vals)
