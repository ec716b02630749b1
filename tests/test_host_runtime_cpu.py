"""Host code of the library on a HIP runtime without a device (fake_hip.c):
which copies, allocations and waits its entry points make.  Each test runs in a
process of its own (runs without a GPU)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, os, sys
sys.path.insert(0, {root!r})
import numpy as np
hip = ctypes.CDLL({fake!r}, mode=ctypes.RTLD_GLOBAL)
import paper_2201_07498_amd as lz
L = lz.lib()
for f in ("fake_used", "fake_idle"): getattr(hip, f).restype = ctypes.c_size_t
hip.fake_count.restype = ctypes.c_long
hip.fake_capacity.argtypes = [ctypes.c_size_t]
hip.fake_pin.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
MB = 1 << 20
D = ctypes.c_void_p(4096)                  # device addresses are never followed
def stream(device=0): return ctypes.c_void_p((77 << 8) + 1 + device)
def spmv(n=1000, nnz=5000, s=None): return L.lz_spmv(D, D, D, n, nnz, 0, D, D, s)
def solve_async(n, nnz, s=None, opt=None):
    return L.lanczos_topk_async(D, D, D, n, nnz, 2, 8, 0, s, D, D, opt, None)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "fake_hip.c"),
                    "-lpthread"], check=True)
    return out


def run(fake, body):
    code = PRELUDE.format(root=ROOT, fake=fake) + body
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout


HOST_SOLVE = """
n, nnz = 2, 8 * 1024 - 2                   # eight whole tiles
rp = np.array([0, nnz // 2, nnz], np.int64)
col, val = np.zeros(nnz, np.int32), np.zeros(nnz, np.float64)
short_col, short_val = {short}
hip.fake_pin(col.ctypes.data, col.nbytes - short_col)
hip.fake_pin(val.ctypes.data, val.nbytes - short_val)
rc = L.lanczos_topk_host(rp.ctypes.data, col.ctypes.data, val.ctypes.data, n, 1, 2, 0, 2048, 0, None, D, D,
                         None, None)
print(rc, hip.fake_count(2))
"""


@pytest.mark.parametrize("short", [(0, 0), (4, 0), (0, 8), (8192, 8192)])
def test_host_arrays_past_their_pinned_allocation_go_through_the_runtime(fake, short):
    # The copy kernel reads the caller's arrays at their host addresses, so it may
    # only be used where they lie inside their pinned allocations as a whole; the
    # runtime's copies check their range and refuse one that does not.
    rc, copies = map(int, run(fake, HOST_SOLVE.format(short=short)).split())
    if short == (0, 0):
        assert copies == 0
    else:
        assert copies > 0 and rc == -3     # LZ_ERR_HIP


def test_workspace_comes_from_the_device_of_the_stream(fake):
    # The current device is 0; the streams belong to devices 0 and 1 and, the default
    # ones (null, legacy, per thread), to the current device.
    out = run(fake, """
for s in (stream(0), stream(1), None, ctypes.c_void_p(1), ctypes.c_void_p(2)):
    assert spmv(s=s) == 0 and solve_async(4000, 20000, s) == 0
print(hip.fake_count(4))
""")
    assert int(out) == 0


FILL = """
# A dozen solves of about 200 MB on streams of their own: idle memory stays with the pool.
streams = [ctypes.c_void_p((k << 8) + 1) for k in range(1, 13)]
for s in streams: assert solve_async(400_000, 1_000_000, s) == 0
for s in streams[1:]: hip.hipStreamSynchronize(s)      # the first stream's free is still pending
idle = hip.fake_idle()
assert idle > 1024 * MB and idle == hip.fake_used()
"""


@pytest.mark.parametrize("call", [
    "solve_async(4_000_000, 40_000_000, streams[0])",                        # past the pool's largest block
    "solve_async(1_000_000, 10_000_000, streams[0])",                        # from the pool, in a larger block than any idle
    "lz.lib().lz_ortho_loss(D, 4096, 4096, 8, 0, None, ctypes.byref(ctypes.c_double()))",
    "lz._server_lib().lz_server_create(0, 900 * MB, 1, 0, ctypes.byref(ctypes.c_void_p()))",
])
def test_idle_pool_memory_is_given_back_before_an_allocation_fails(fake, call):
    # The call's memory is there only together with what the pool keeps idle.
    need = int(run(fake, f"""
streams = [stream()]
assert {call} == 0
print(hip.fake_used(), flush=True)
os._exit(0)
"""))
    for lag in (0, 3):             # the driver may have given-back memory a little later
        run(fake, FILL + f"""
hip.fake_lag({lag})
hip.fake_capacity(max(idle, {need}) + 8 * MB)
assert {call} == 0
os._exit(0)
""")


def test_allocation_fails_cleanly_where_giving_back_is_not_enough(fake):
    run(fake, FILL + """
hip.fake_capacity(idle + 8 * MB)
assert solve_async(40_000_000, 400_000_000, streams[0]) == -2     # LZ_ERR_OUT_OF_MEMORY
assert solve_async(4000, 20000, streams[0]) == 0
""")


def test_no_wait_and_no_pool_inside_a_capture(fake):
    # An allocation inside a capture is a graph node: it goes to the default pool,
    # and one that fails is refused without waiting for the stream.
    run(fake, """
hip.fake_capturing(1)
assert solve_async(4000, 20000, stream()) == 0 and hip.fake_idle() == hip.fake_used() > 0
idle = hip.fake_idle()
hip.fake_capacity(idle + 8 * MB)
assert solve_async(4_000_000, 40_000_000, stream()) == -2 and hip.fake_idle() == idle
""")


def test_release_memory_gives_back_what_is_idle(fake):
    run(fake, FILL + """
lz.release_memory()
pending = hip.fake_used()
assert 0 < pending < idle // 4                       # the first stream has yet to free its block
hip.hipStreamSynchronize(streams[0])
lz.release_memory()
assert hip.fake_used() == 0
assert solve_async(4000, 20000, stream()) == 0 and hip.fake_used() > 0
""")


def test_pinned_buffers_do_not_pile_up_with_threads(fake):
    # One buffer serves calls in any number of threads that do not overlap, and
    # overlapping ones take no more than one each.
    run(fake, """
import threading
def work():
    assert spmv(s=stream()) == 0
    lz.tridiag_eig(np.ones(4), np.ones(3))
    L.lanczos_topk_ex(D, D, D, 1000, 5000, 2, 8, 0, stream(), D, D, None, None)
for _ in range(20):
    t = threading.Thread(target=work); t.start(); t.join()
assert hip.fake_count(1) == 1, hip.fake_count(1)
ts = [threading.Thread(target=work) for _ in range(40)]
for t in ts: t.start()
for t in ts: t.join()
assert hip.fake_count(1) <= 40
n = hip.fake_count(0)
work()
assert hip.fake_count(0) == n
""")
