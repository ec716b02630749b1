"""Calls on the default stream's handles (null, legacy, per thread) and on a stream
of their own give the same bits."""
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402
import synth  # noqa: E402
from gpu_util import device_csr  # noqa: E402

pytestmark = pytest.mark.gpu


class Handle:
    def __init__(self, value):
        self.cuda_stream = value


@pytest.mark.parametrize("handle", [0, 1, 2, None])
def test_default_stream_handles(handle):
    csr = device_csr(*synth.er(3000, 6.0, seed=2), "fp64")
    x = torch.rand(3000, dtype=torch.float64, device="cuda:0")
    want = lz.topk(*csr, 4, 12, "fp64", seed=5), lz.spmv(*csr, x)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if handle is None else Handle(handle)
    vals, vecs, _ = lz.topk(*csr, 4, 12, "fp64", seed=5, stream=stream)
    y = lz.spmv(*csr, x, stream=stream)
    loss = lz.ortho_loss(vecs, "fp64", stream=stream)
    torch.cuda.synchronize()
    b = lz.topk_async(*csr, 4, 12, "fp64", seed=5, stream=stream)
    torch.cuda.synchronize()
    assert torch.equal(vals, want[0][0]) and torch.equal(vecs, want[0][1]) and torch.equal(y, want[1])
    assert torch.equal(vals, b[0]) and torch.equal(vecs, b[1]) and loss < 1e-12
