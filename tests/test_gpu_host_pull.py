"""Slab copies from pinned host arrays that start anywhere within 16 bytes, from a
few entries to many slabs: bit for bit the device-resident solve."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2201_07498_amd as lz  # noqa: E402
import synth  # noqa: E402
from gpu_util import device_csr  # noqa: E402

pytestmark = pytest.mark.gpu
DT = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}


def pinned_at(t, offset):
    """A pinned copy of t whose first element is `offset` elements into its allocation."""
    buf = torch.empty(t.numel() + offset, dtype=t.dtype, pin_memory=True)
    buf[offset:] = t
    return buf[offset:]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("offset", [0, 1, 2, 3, 5, 7])
@pytest.mark.parametrize("n", [2, 5, 1500, 40_001])
def test_slabs_from_unaligned_host_arrays(precision, offset, n):
    rp, c, v = synth.er(n, min(9.0, n / 2), seed=n + offset)
    v = synth.round_values(v, precision)
    K, m = min(2, n), min(6, n)
    col = torch.from_numpy(np.ascontiguousarray(c, dtype=np.int32))
    val = torch.from_numpy(np.ascontiguousarray(v, dtype=np.float64)).to(DT[precision])
    got = lz.topk_host(torch.from_numpy(rp), pinned_at(col, offset), pinned_at(val, offset), K, m, precision,
                       slab_nnz=2048 + 37 * offset, seed=3)
    want = lz.topk(*device_csr(rp, c, v, precision), K, m, precision, seed=3, reorder="off")
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
