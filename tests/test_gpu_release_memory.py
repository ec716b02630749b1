"""Device memory that the library keeps between calls is bounded and can be given back."""
import time

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

    def release(target=None):
        # The driver has the memory when the runtime has dropped its last references,
        # on a thread of its own.
        lz.release_memory()
        end = time.monotonic() + 2.0
        while True:
            time.sleep(0.05)
            free = torch.cuda.mem_get_info()[0]
            if target is None or free >= target or time.monotonic() > end:
                return free

    solve()                                   # code objects, streams and scratch of the first call
    before = release()
    kept = before - solve()
    vals = out[0].clone()
    need = lz.workspace_size(200_000, csr[1].numel(), 8, 24, "fp64")
    print(f"workspace {need} bytes, kept {kept}", flush=True)
    assert need // 2 < kept <= 2 << 30
    assert release(before) >= before
    solve()
    assert torch.equal(out[0], vals)
