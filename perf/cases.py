"""The solves and component calls whose speed this library is measured by.

Every case is a plain dict; `prepare` makes its inputs on the GPU from a seed,
`run` is one pass through the public entry points of `paper_2201_07498_amd`,
and `exact` computes the same outputs in binary64 with torch and numpy alone.

Kinds of case (`kind`):
  solve    topk or topk_async on a device-resident CSR matrix
  server   a burst of requests through Server (continuous batching)
  host     topk_host: entries in pinned host memory, streamed to the device
  spmv     one y = A x
  tridiag  one tridiagonal Jacobi eigensolve

Matrices are the seeded synthetic ones of the benchmark: Erdos-Renyi with a
full diagonal, and R-MAT with (a, b, c, d) = (0.57, 0.19, 0.19, 0.05),
symmetrised and deduplicated, U(0, 1) weights, optionally normalised to
D^-1/2 A D^-1/2.
"""
import math

import numpy as np
import torch

import paper_2201_07498_amd as lz

DEV = "cuda:0"
DTYPE = {"fp64": torch.float64, "fp32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"fp64": 8, "fp32": 4, "bf16": 2}


def _solve(name, graph, n, degree, K, m, precision, **kw):
    """degree: mean number of entries per row (R-MAT: of draws, before
    duplicates are dropped)."""
    case = dict(name=name, kind="solve", graph=graph, n=n, degree=degree, K=K, m=m, precision=precision,
                normalise=False, entry="topk", reorth="twice", arith="mixed", workspace=False)
    case.update(kw)
    return case


def listed():
    return [
        # The smallest calls: a few thousand rows, where launches and latency are all there is.
        _solve("er3k_fp64", "er", 3000, 10.0, 4, 16, "fp64"),
        # The paper-sized small workload of the benchmark, called as a pipelined service calls it (stream-ordered,
        # workspace kept).
        _solve("er10k_fp64_async", "er", 10_000, 10.0, 8, 24, "fp64", entry="topk_async", workspace=True),
        # An ordinary request of the serving mix solved alone: ragged n, power-law rows, relabelled by the solver.
        _solve("rmat150k_fp64", "rmat", 150_001, 16.0, 16, 48, "fp64"),
        # Uniform random rows (never relabelled): gathers without locality, FP32 storage.
        _solve("er500k_fp32", "er", 500_009, 18.0, 8, 24, "fp32"),
        # R-MAT scale 20, edge factor 8, normalised: the benchmark's mid-size workload in its precisions.
        _solve("rmat20_fp32", "rmat", 1 << 20, 16.0, 16, 48, "fp32", normalise=True, workspace=True),
        _solve("rmat20_fp64", "rmat", 1 << 20, 16.0, 16, 48, "fp64", workspace=True),
        # R-MAT scale 23, edge factor 16 in BF16 storage, the benchmark's 16-bit workload.
        _solve("rmat23_bf16", "rmat", 1 << 23, 32.0, 24, 64, "bf16", workspace=True),
        # The largest: R-MAT edge factor 16 with K = 8, m = 32, half the rows of the benchmark's scale 26, so that a
        # state fits the card three times over.
        _solve("rmat25_fp32", "rmat", 1 << 25, 32.0, 8, 32, "fp32", workspace=True),
        # A burst of queued requests over a pool of matrices in pinned host memory, precisions mixed.
        dict(name="server_mix", kind="server", requests=16, slots=8, n_min=12_000, n_max=1_000_000),
        # A matrix whose entries stay in host memory, half of them resident.
        dict(name="host_rmat19_fp32", kind="host", graph="rmat", n=1 << 19, degree=16.0, K=8, m=24,
             precision="fp32", normalise=False, slab=1 << 20, resident=0.5),
        # The component entry points.
        dict(name="spmv_er1m_fp32", kind="spmv", graph="er", n=1_000_003, degree=16.0, precision="fp32",
             normalise=False),
        dict(name="tridiag_m64", kind="tridiag", m=64),
    ]


def draw(rng):
    """One more case of the listed ranges: sizes over their logarithm, ragged,
    every precision, entry point and option that is used in earnest."""
    kind = rng.choices(["solve", "server", "host", "spmv", "tridiag"], [0.72, 0.06, 0.06, 0.1, 0.06])[0]
    if kind == "tridiag":
        return dict(kind="tridiag", m=rng.randint(8, 64))
    if kind == "server":
        return dict(kind="server", requests=rng.randint(8, 16), slots=rng.choice([2, 4, 8]), n_min=12_000,
                    n_max=int(math.exp(rng.uniform(math.log(1e5), math.log(1e6)))))
    n = int(math.exp(rng.uniform(math.log(2000), math.log(1 << 21))))
    graph = rng.choice(["er", "rmat"])
    degree = round(rng.uniform(4.0, 32.0), 2)
    precision = rng.choice(["fp64", "fp32", "bf16"])
    if kind == "spmv":
        return dict(kind="spmv", graph=graph, n=n, degree=degree, precision=precision, normalise=False)
    K = rng.choice([4, 8, 16])
    m = 3 * K
    if kind == "host":
        return dict(kind="host", graph=graph, n=min(n, 1 << 19), degree=degree, K=K, m=m, precision=precision,
                    normalise=False, slab=1 << 20, resident=rng.choice([0.0, 0.5]))
    case = _solve("", graph, n, degree, K, m, precision, entry=rng.choice(["topk", "topk", "topk_async"]),
                  workspace=rng.random() < 0.5, reorth=rng.choice(["twice", "twice", "twice", "once", "selective"]))
    if precision == "fp32" and rng.random() < 0.25:
        case["arith"] = "fp32"
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _pairs_er(n, degree, g):
    """Unordered vertex pairs, uniform, as sorted keys lo * n + hi (lo < hi)."""
    count = int(n * (degree - 1.0) / 2.0)
    a = torch.randint(0, n, (count,), device=DEV, generator=g)
    b = torch.randint(0, n, (count,), device=DEV, generator=g)
    return _unique_pairs(a, b, n)


def _pairs_rmat(n, degree, g):
    """R-MAT draws over the next power of two (those past n dropped), vertex
    ids permuted."""
    scale = max(1, math.ceil(math.log2(n)))
    left = int(n * degree / 2.0)
    perm = torch.randperm(n, device=DEV, generator=g)
    parts = []
    while left > 0:                                  # in pieces, for the memory of the largest matrices
        count = min(left, 1 << 27)
        left -= count
        a = torch.zeros(count, dtype=torch.int32, device=DEV)
        b = torch.zeros(count, dtype=torch.int32, device=DEV)
        for _ in range(scale):
            r = torch.rand(count, device=DEV, generator=g)
            a = a * 2 + (r >= 0.76)
            b = b * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
            del r
        if n < (1 << scale):
            keep = (a < n) & (b < n)
            a, b = a[keep], b[keep]
        a, b = perm[a.long()], perm[b.long()]
        parts.append(_unique_pairs(a, b, n))
        del a, b
    if len(parts) == 1:
        return parts[0]
    keys = torch.cat(parts)
    del parts
    return _unique_sorted(keys.sort().values)


def _unique_sorted(keys):
    keep = torch.ones(keys.numel(), dtype=torch.bool, device=keys.device)
    torch.ne(keys[1:], keys[:-1], out=keep[1:])
    return keys[keep]


def _unique_pairs(a, b, n):
    lo, hi = torch.minimum(a, b), torch.maximum(a, b)
    keys = (lo * n + hi)[lo != hi]
    return _unique_sorted(keys.sort().values)


def _matrix(case, seed):
    """(rowptr, col, val): int64, int32 and the storage type, on the GPU."""
    g = _generator(seed)
    n, er = case["n"], case["graph"] == "er"
    keys = _pairs_er(n, case["degree"], g) if er else _pairs_rmat(n, case["degree"], g)
    pairs = keys.numel()
    w = torch.rand(pairs, device=DEV, generator=g)
    if er:
        w = w * 2.0 - 1.0
    lo = torch.div(keys, n, rounding_mode="floor")
    hi = keys - lo * n
    del keys
    both = [lo * n + hi, hi * n + lo]
    del lo, hi
    if er:
        both.append(torch.arange(n, device=DEV) * (n + 1))
    both = torch.cat(both)
    both, order = both.sort()
    row = torch.div(both, n, rounding_mode="floor")
    col = (both - row * n).to(torch.int32)
    del both
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(row, minlength=n), 0, out=rowptr[1:])
    if er:
        w = torch.cat([w, w, torch.rand(n, device=DEV, generator=g)])
        val = w[order]
    else:
        order = torch.where(order >= pairs, order - pairs, order)
        val = w[order]
    del w, order
    if case["normalise"]:
        d = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, row, val.double())
        s = torch.where(d > 0, d.rsqrt(), d)
        val = (val.double() * s[row] * s[col.long()]).float()
    return rowptr, col, val.to(DTYPE[case["precision"]])


def _server_pool(case, seed):
    """The burst: matrices of log-spaced sizes in pinned host memory, and the
    requests (matrix, K, m, precision, seed) over them."""
    rng = np.random.default_rng(seed)
    kinds = np.random.default_rng(3)                 # the same shapes and precisions for every seed
    pool = []
    count = 6
    for i in range(count):
        n = int(case["n_min"] * (case["n_max"] / case["n_min"]) ** (i / (count - 1))) + int(rng.integers(100))
        spec = dict(graph="rmat" if i % 2 else "er", n=n, degree=float(rng.uniform(4.0, 24.0)), precision="fp32",
                    normalise=False)
        rp, col, val = _matrix(spec, seed * 64 + i)
        pool.append(dict(rp=rp.cpu().pin_memory(), col=col.cpu().pin_memory(),
                         **{p: val.to(DTYPE[p]).cpu().pin_memory() for p in DTYPE}))
    requests = []
    for i in range(case["requests"]):
        K = int(kinds.choice([4, 8, 16]))
        requests.append((int(i % count), K, 3 * K, str(kinds.choice(["fp64", "fp32", "bf16"])), i))
    return pool, requests


class _Serving:
    """A server and the burst it is sent; closed with the state."""

    def __init__(self, case, seed):
        self.pool, self.requests = _server_pool(case, seed)
        self.server = lz.Server(24 << 30, max_slots=case["slots"])

    def __del__(self):
        server = getattr(self, "server", None)
        if server is not None:
            server.close()


def _tridiag(case, seed):
    """alpha and beta as a Lanczos run on a random matrix gives them."""
    rng = np.random.default_rng(seed)
    m = case["m"]
    return rng.normal(0.0, 0.3, m), 1.0 + 0.2 * rng.random(m - 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "tridiag":
        alpha, beta = _tridiag(case, seed)
        return dict(case=case, alpha=alpha, beta=beta)
    if kind == "server":
        return dict(case=case, serving=_Serving(case, seed))
    rp, col, val = _matrix(case, seed)
    st = dict(case=case, seed=int(seed), rp=rp, col=col, val=val)
    n, nnz = case["n"], col.numel()
    if kind == "spmv":
        st["x"] = torch.rand(n, device=DEV, generator=_generator(seed + 1)).to(val.dtype)
    elif kind == "host":
        st.update(rp=rp.cpu(), col=col.cpu().pin_memory(), val=val.cpu().pin_memory(),
                  resident=int(case["resident"] * nnz))
    elif case["workspace"]:
        size = lz.workspace_size(n, nnz, case["K"], case["m"], case["precision"])
        st["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
        st["out"] = (torch.empty(case["K"], dtype=torch.float64, device=DEV),
                     torch.empty(case["K"], n, dtype=torch.float64, device=DEV))
    return st


# --------------------------------------------------------------------- run
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "tridiag":
        theta, S, _ = lz.tridiag_eig(st["alpha"], st["beta"])
        return dict(theta=theta, S=S)
    if kind == "server":
        sv = st["serving"]
        tickets = []
        for which, K, m, prec, seed in sv.requests:
            p = sv.pool[which]
            tickets.append(sv.server.submit(p["rp"], p["col"], p[prec], K, m, prec, seed=seed))
        got = []
        for t in tickets:
            vals, _, res = sv.server.wait(t)
            sv.server.release(t)
            got.append(dict(vals=vals, resid=res["resid"]))
        return got
    if kind == "spmv":
        return lz.spmv(st["rp"], st["col"], st["val"], st["x"], case["precision"])
    if kind == "host":
        vals, vecs, rep = lz.topk_host(st["rp"], st["col"], st["val"], case["K"], case["m"], case["precision"],
                                       slab_nnz=case["slab"], resident_nnz=st["resident"], seed=st["seed"])
        return dict(vals=vals, vecs=vecs, resid=rep["resid"])
    kw = dict(seed=st["seed"], reorth=case["reorth"], arith=case["arith"])
    if case["workspace"]:
        kw.update(workspace=st["ws"], out=st["out"])
    args = (st["rp"], st["col"], st["val"], case["K"], case["m"], case["precision"])
    if case["entry"] == "topk_async":
        vals, vecs, _ = lz.topk_async(*args, **kw)
        return dict(vals=vals, vecs=vecs)
    vals, vecs, rep = lz.topk(*args, **kw)
    return dict(vals=vals, vecs=vecs, resid=rep["resid"])


# -------------------------------------------------------------------- work
def _entries(case):
    n, d = case["n"], case["degree"]
    return n * d                                     # duplicates that were dropped are not taken off


def _solve_work(n, z, K, m, precision):
    """Per step: the matrix and v read, w written and read, the basis read
    twice (dots, update) and one column written; then the Ritz product (basis
    read, n x K written), one product with all Ritz vectors, and the outputs."""
    vb = BYTES[precision]
    wb = 8 if precision == "fp64" else 4
    mat = z * (4 + vb) + 8.0 * n
    steps = m * (mat + n * (2.0 * vb + 3.0 * wb)) + n * vb * float(m * (m + 1))
    finish = n * m * vb * 2.0 + mat + 8.0 * n * K * 3
    flops = m * (2.0 * z) + 4.0 * n * m * (m + 1) / 2 + 2.0 * n * m * K + 2.0 * z * K + 2.0 * n * (m * m + K * K)
    return dict(bytes=steps + finish, flops=flops)


def work(case):
    kind = case["kind"]
    if kind == "tridiag":
        m = case["m"]
        return dict(bytes=8.0 * (2 * m + m * m + m), flops=8.0 * 6.0 * m ** 3)
    if kind == "server":
        total = dict(bytes=0.0, flops=0.0)
        for i in range(case["requests"]):
            n = case["n_min"] * (case["n_max"] / case["n_min"]) ** ((i % 6) / 5)
            w = _solve_work(n, 14.0 * n, 8, 24, "fp32")
            total = {k: total[k] + w[k] for k in total}
        return total
    n, z = case["n"], _entries(case)
    if kind == "spmv":
        vb = BYTES[case["precision"]]
        return dict(bytes=z * (4 + vb) + 8.0 * n + n * (vb + (8 if vb == 8 else 4)), flops=2.0 * z)
    return _solve_work(n, z, case["K"], case["m"], case["precision"])


# ------------------------------------------------------------------- exact
def _u01(seed, n):
    """U01 of the SplitMix64 stream started at `seed` (int64 arithmetic wraps)."""
    def shr(z, k):
        return (z >> k) & ((1 << (64 - k)) - 1)

    def signed(c):
        return c - (1 << 64) if c >= (1 << 63) else c
    z = torch.arange(1, n + 1, dtype=torch.int64, device=DEV) * signed(0x9E3779B97F4A7C15) + int(seed)
    z = (z ^ shr(z, 30)) * signed(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * signed(0x94D049BB133111EB)
    return shr(z ^ shr(z, 31), 11).double() * 2.0 ** -53


def _exact_solve(rp, col, val, K, m, seed):
    """Krylov Rayleigh-Ritz in binary64: Lanczos with two Gram-Schmidt passes,
    a dense eigensolve of T, the K Ritz pairs of largest modulus."""
    n = rp.numel() - 1
    A = torch.sparse_csr_tensor(rp.to(torch.int32), col, val.double(), (n, n))
    V = torch.zeros(m, n, dtype=torch.float64, device=DEV)
    u = _u01(seed, n)
    V[0] = u / u.norm()
    alpha, beta = np.zeros(m), np.zeros(m)
    for j in range(m):
        w = A @ V[j]
        alpha[j] = float(w @ V[j])
        for _ in range(2):
            w = w - (V[: j + 1] @ w) @ V[: j + 1]
        beta[j] = float(w.norm())
        if j + 1 < m:
            V[j + 1] = w / beta[j]
    theta, S = np.linalg.eigh(np.diag(alpha) + np.diag(beta[:-1], 1) + np.diag(beta[:-1], -1))
    top = np.lexsort((-theta, -np.abs(theta)))[:K]
    Y = torch.from_numpy(np.ascontiguousarray(S[:, top].T)).to(DEV) @ V
    del V
    Y = Y / Y.norm(dim=1, keepdim=True)
    big = Y.gather(1, Y.abs().argmax(dim=1, keepdim=True))
    Y = Y * torch.where(big < 0, -1.0, 1.0)
    lam = torch.from_numpy(theta[top].copy()).to(DEV)
    resid = torch.stack([(A @ Y[k] - lam[k] * Y[k]).norm() / lam[k].abs() for k in range(K)])
    return lam, Y.T, resid


def exact(case, seed):
    kind = case["kind"]
    if kind == "tridiag":
        return None                                  # Jacobi order and signs of the columns are the method's own
    if kind == "server":
        pool, requests = _server_pool(case, seed)
        got = []
        for which, K, m, prec, s in requests:
            p = pool[which]
            if prec == "bf16":                       # the storage's rounding moves unconverged pairs, and their order
                got.append(dict(vals=None, resid=None))
                continue
            lam, _, resid = _exact_solve(p["rp"].to(DEV), p["col"].to(DEV), p[prec].to(DEV), K, m, s)
            got.append(dict(vals=lam, resid=resid))
        return got
    if kind != "spmv" and case["precision"] == "bf16":
        return None                                  # the storage's rounding moves unconverged pairs, and their order
    rp, col, val = _matrix(case, seed)
    if kind == "spmv":
        x = torch.rand(case["n"], device=DEV, generator=_generator(seed + 1)).to(val.dtype)
        A = torch.sparse_csr_tensor(rp.to(torch.int32), col, val.double(), (case["n"], case["n"]))
        return A @ x.double()
    lam, Y, resid = _exact_solve(rp, col, val, case["K"], case["m"], seed)
    if kind == "solve" and case["entry"] == "topk_async":
        return dict(vals=lam, vecs=Y)
    return dict(vals=lam, vecs=Y, resid=resid)
