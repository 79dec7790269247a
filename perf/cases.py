"""Workloads of the library as its users call it, for timing.

Every case goes through the public entry points of ``paper_2001_07938_amd``:
the paper-shaped call on host arrays, products on a device-resident handle,
a grouped batch, the conjugate gradient and PageRank loops, BFS, the dot
product and the JDS product.  The matrices are those of the benchmark and the
tests (rows of uniformly random columns, 3D stencils, a strictly diagonally
dominant random matrix, R-MAT graphs), drawn here on the device from a seed.

``listed()`` names the cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare(case, seed)`` makes inputs and handles, ``run(state)`` is one
pass, ``work(case)`` what a pass cannot do without, ``exact(case, seed)`` the
same result from plain torch in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2001_07938_amd as lilac

DEVICE = "cuda"
DAMPING = 0.85


def listed():
    return [
        # the call the paper's compiler inserts in place of the source loop:
        # host arrays, matrix resident after the first call, x sent and y
        # returned on every call (the benchmark's spmv16 size)
        dict(name="raw_host_4096", op="raw", kind="uniform", n=4096, per_row=16, dtype="f64"),
        # the smallest product on a handle: launch latency counts
        dict(name="spmv_uniform_4096", op="spmv", kind="uniform", n=4096, per_row=16, dtype="f64"),
        # one unstructured matrix of ordinary size, 5 to 60 entries per row
        dict(name="spmv_random_200k", op="spmv", kind="random", n=200_000, lo=5, hi=60, dtype="f64"),
        # a graph's adjacency as it comes: scattered hubs, empty rows and
        # rows of tens of thousands of entries, float32
        dict(name="spmv_rmat_20_f32", op="spmv", kind="rmat", scale=20, edges=1 << 24, dtype="f32"),
        # a large 27-point stencil, float64
        dict(name="spmv_stencil27_128", op="spmv", kind="stencil", k=128, points=27, dtype="f64"),
        # the NPB-CG stand-in of the benchmark: 75 iterations, one graph
        dict(name="cg_spd_150k", op="cg", kind="spd", n=150_000, half=120, iters=75),
        # a small solve (the request server's kind): latency of an iteration
        dict(name="cg_stencil7_32", op="cg", kind="stencil", k=32, points=7, iters=50),
        # PageRank over the benchmark's graph size
        dict(name="pagerank_rmat_22", op="pagerank", kind="rmat", scale=22, edges=1 << 26, iters=20),
        # the benchmark's batch: 512 matrices, a third each of 7-point
        # stencils, 27-point stencils and random rows, one call
        dict(name="batched_512", op="batched", count=512, n_lo=1000, n_hi=200_000, sizes=20010797,
             dtype="f64"),
        # breadth-first search levels over a graph
        dict(name="bfs_rmat_20", op="bfs", kind="rmat", scale=20, edges=1 << 24),
        # the dense dot product, memory bound
        dict(name="dot_f64_64m", op="dot", n=1 << 26, dtype="f64"),
        # the second format: JDS arrays on the device, as converted from CSR
        dict(name="jds_random_200k", op="jds", kind="random", n=200_000, lo=5, hi=60),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes spread over the ranges of the listed ones (by
    their logarithm), odd ones among them, both value types where the entry
    point takes them."""
    op = rng.choice(["raw", "spmv", "spmv", "spmv", "cg", "pagerank", "batched", "bfs", "dot", "jds"])
    dtype = rng.choice(["f64", "f32"])
    if op == "raw":
        return dict(op=op, kind="uniform", n=_log_uniform(rng, 500, 50_000),
                    per_row=rng.randint(3, 40), dtype=dtype)
    if op == "spmv":
        kind = rng.choice(["uniform", "random", "rmat", "stencil"])
        if kind == "uniform":
            return dict(op=op, kind=kind, n=_log_uniform(rng, 1000, 100_000),
                        per_row=rng.randint(3, 60), dtype=dtype)
        if kind == "random":
            return dict(op=op, kind=kind, n=_log_uniform(rng, 20_000, 500_000), lo=5,
                        hi=rng.randint(20, 120), dtype=dtype)
        if kind == "rmat":
            scale = rng.randint(14, 21)
            return dict(op=op, kind=kind, scale=scale,
                        edges=int((1 << scale) * rng.uniform(6.0, 24.0)), dtype=dtype)
        return dict(op=op, kind=kind, k=_log_uniform(rng, 20, 160), points=rng.choice([7, 27]),
                    dtype=dtype)
    if op == "cg":
        if rng.random() < 0.5:
            return dict(op=op, kind="spd", n=_log_uniform(rng, 5000, 150_000),
                        half=rng.randint(10, 120), iters=rng.randint(20, 75))
        return dict(op=op, kind="stencil", k=_log_uniform(rng, 10, 100), points=rng.choice([7, 27]),
                    iters=rng.randint(20, 75))
    if op in ("pagerank", "bfs"):
        scale = rng.randint(13, 21)
        edges = int((1 << scale) * rng.uniform(6.0, 20.0))
        if op == "bfs":
            return dict(op=op, kind="rmat", scale=scale, edges=edges)
        return dict(op=op, kind="rmat", scale=scale, edges=edges, iters=rng.randint(5, 30))
    if op == "batched":
        return dict(op=op, count=_log_uniform(rng, 16, 400), n_lo=1000, n_hi=200_000,
                    sizes=rng.randint(1, 1 << 30), dtype=dtype)
    if op == "dot":
        return dict(op=op, n=_log_uniform(rng, 1000, 1 << 26), dtype=dtype)
    return dict(op=op, kind="random", n=_log_uniform(rng, 2000, 400_000), lo=rng.randint(1, 5),
                hi=rng.randint(20, 120))


# ------------------------------------------------------------------ matrices

def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.float64


def _uniform(n, g, dtype):
    return torch.rand(n, generator=g, device=DEVICE, dtype=dtype) * 2 - 1


def _row_ptr(rows, counts):
    rp = torch.zeros(rows + 1, dtype=torch.int64, device=DEVICE)
    torch.cumsum(counts, 0, out=rp[1:])
    return rp.to(torch.int32)


def _from_keys(rows, cols, key, vals):
    """CSR arrays of entries at the ascending keys row * cols + col."""
    r = torch.div(key, cols, rounding_mode="floor")
    c = (key - r * cols).to(torch.int32)
    return _row_ptr(rows, torch.bincount(r, minlength=rows)), c, vals


def _random_rows(n, lo, hi, g, dtype):
    """lo to hi distinct uniformly random columns per row, values U[-1, 1)."""
    cnt = torch.randint(lo, hi + 1, (n,), generator=g, device=DEVICE)
    r = torch.repeat_interleave(torch.arange(n, device=DEVICE), cnt)
    c = torch.randint(0, n, (r.numel(),), generator=g, device=DEVICE)
    key = torch.unique(r * n + c)
    return _from_keys(n, n, key, _uniform(key.numel(), g, dtype))


def _stencil(k, points, dtype):
    """3D stencil on a k^3 grid, Dirichlet truncation: the diagonal is the
    number of neighbours, each neighbour -1."""
    n = k ** 3
    span = (-1, 0, 1)
    offs = [(z, y, x) for z in span for y in span for x in span
            if points == 27 or abs(z) + abs(y) + abs(x) <= 1]
    i = torch.arange(n, device=DEVICE, dtype=torch.int32)
    z, y, x = i // (k * k), (i // k) % k, i % k
    col = torch.empty((n, len(offs)), dtype=torch.int32, device=DEVICE)
    ok = torch.empty((n, len(offs)), dtype=torch.bool, device=DEVICE)
    for t, (dz, dy, dx) in enumerate(offs):
        col[:, t] = i + (dz * k * k + dy * k + dx)
        ok[:, t] = ((z + dz >= 0) & (z + dz < k) & (y + dy >= 0) & (y + dy < k)
                    & (x + dx >= 0) & (x + dx < k))
    vals = torch.full((n, len(offs)), -1.0, dtype=dtype, device=DEVICE)
    vals[:, offs.index((0, 0, 0))] = float(points - 1)
    return _row_ptr(n, ok.sum(1)), col[ok], vals[ok]


def _spd(n, half, g):
    """Symmetric, strictly diagonally dominant: `half` random partners per row,
    one U[-1, 1) value for each distinct pair, diagonal sum |a_ij| + 1."""
    i = torch.repeat_interleave(torch.arange(n, device=DEVICE), half)
    j = (i + 1 + torch.randint(0, n - 1, (i.numel(),), generator=g, device=DEVICE)) % n
    key = torch.unique(torch.minimum(i, j) * n + torch.maximum(i, j))
    lo = torch.div(key, n, rounding_mode="floor")
    hi = key - lo * n
    v = _uniform(key.numel(), g, torch.float64)
    # sums of |a_ij| in fixed point, so that their order does not matter
    fixed = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    q = (v.abs() * (1 << 30)).to(torch.int64) + 1
    fixed.index_add_(0, lo, q)
    fixed.index_add_(0, hi, q)
    diag = fixed.to(torch.float64) / (1 << 30) + 1.0
    d = torch.arange(n, device=DEVICE)
    full, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo, d * n + d]))
    return _from_keys(n, n, full, torch.cat([v, v, diag])[order])


def _rmat(scale, edges, g, dtype):
    """Pull-direction CSR of an R-MAT graph (0.57, 0.19, 0.19, 0.05): vertices
    renamed by a random permutation, duplicate edges removed, the value of
    edge u -> v at (v, u) is 1 / outdeg(u)."""
    nv = 1 << scale
    src = torch.zeros(edges, dtype=torch.int64, device=DEVICE)
    dst = torch.zeros(edges, dtype=torch.int64, device=DEVICE)
    for _ in range(scale):
        u = torch.rand(edges, generator=g, device=DEVICE)
        src = (src << 1) | (u >= 0.76)
        dst = (dst << 1) | (((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    perm = torch.randperm(nv, generator=g, device=DEVICE)
    key = torch.unique((perm[dst] << scale) | perm[src])
    del src, dst
    c = key & (nv - 1)
    w = (1.0 / torch.bincount(c, minlength=nv)[c].to(torch.float64)).to(dtype)
    return _from_keys(nv, nv, key, w)


def _matrix(case, g):
    """(row_ptr, col_idx, vals) on the device."""
    dt = torch.float32 if case["op"] in ("pagerank", "bfs") else _dtype(case)
    kind = case["kind"]
    if kind == "uniform":
        return _random_rows(case["n"], case["per_row"], case["per_row"], g, dt)
    if kind == "random":
        return _random_rows(case["n"], case["lo"], case["hi"], g, dt)
    if kind == "stencil":
        return _stencil(case["k"], case["points"], dt)
    if kind == "spd":
        return _spd(case["n"], case["half"], g)
    return _rmat(case["scale"], case["edges"], g, dt)


def _batch_specs(case):
    """(kind, size) of each matrix: sizes log-uniform, kinds in equal thirds."""
    rng = np.random.default_rng(case["sizes"])
    n = np.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), case["count"]))
    kind = np.array(["st7", "st27", "rand"])[np.arange(case["count"]) % 3]
    rng.shuffle(kind)
    return [(str(t), int(round(m)) if t == "rand" else max(2, round(m ** (1 / 3)))) for t, m in zip(kind, n)]


def _batch_matrix(spec, g, dtype):
    kind, n = spec
    if kind == "rand":
        return _random_rows(n, 5, 60, g, dtype)
    return _stencil(n, 7 if kind == "st7" else 27, dtype)


def _batch_vectors(case, g):
    """x of every matrix in one buffer, each at a multiple of 32 elements."""
    rows = [n if kind == "rand" else n ** 3 for kind, n in _batch_specs(case)]
    at = np.concatenate([[0], np.cumsum([(r + 31) // 32 * 32 for r in rows])])
    return rows, at, _uniform(int(at[-1]), g, _dtype(case))


def _source(case, ci):
    """A vertex with outgoing edges."""
    return int(ci[ci.numel() // 2]) if ci.numel() else 0


# ------------------------------------------------------------ the entry points

def prepare(case, seed):
    op, g, dt = case["op"], _gen(seed), _dtype(case)
    s = dict(case=case)
    if op == "dot":
        s.update(a=_uniform(case["n"], g, dt), b=_uniform(case["n"], g, dt),
                 out=torch.zeros((), dtype=dt, device=DEVICE))
        return s
    if op == "batched":
        s["handles"] = [lilac.Csr(*_batch_matrix(m, g, dt)) for m in _batch_specs(case)]
        rows, at, s["x"] = _batch_vectors(case, g)
        s["y"] = torch.zeros_like(s["x"])
        s["xs"] = [s["x"][a:a + r] for a, r in zip(at, rows)]
        s["ys"] = [s["y"][a:a + r] for a, r in zip(at, rows)]
        return s
    rp, ci, v = _matrix(case, g)
    n = rp.numel() - 1
    if op == "raw":
        s.update(n=n, rp=rp.cpu().numpy(), ci=ci.cpu().numpy(), v=v.cpu().numpy(),
                 x=_uniform(n, g, dt).cpu().numpy(), y=np.zeros(n, np.float32 if dt == torch.float32 else np.float64))
        # new arrays may lie where older ones of this process were cached
        for a in (s["rp"], s["ci"], s["v"]):
            lilac.lilac_invalidate(a)
        return s
    if op == "pagerank":
        s.update(A=lilac.Csr(rp, ci, v, cols=n), x=torch.empty(n, dtype=torch.float32, device=DEVICE))
    elif op == "bfs":
        s.update(A=lilac.Csr(rp, ci, v, cols=n), source=_source(case, ci),
                 level=torch.empty(n, dtype=torch.int32, device=DEVICE))
    elif op == "cg":
        s.update(A=lilac.Csr(rp, ci, v, cols=n), b=_uniform(n, g, torch.float64),
                 x=torch.empty(n, dtype=torch.float64, device=DEVICE))
    elif op == "jds":
        s.update(n=n, J=lilac.Csr(rp, ci, v, cols=n).to_jds(), x=_uniform(n, g, torch.float64),
                 y=torch.empty(n, dtype=torch.float64, device=DEVICE))
    else:
        s.update(A=lilac.Csr(rp, ci, v, cols=n), x=_uniform(n, g, dt),
                 y=torch.empty(n, dtype=dt, device=DEVICE))
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "raw":
        f = lilac.lilac_spmv_csr_f32 if case["dtype"] == "f32" else lilac.lilac_spmv_csr
        return f(s["n"], s["rp"], s["ci"], s["v"], s["x"], s["y"])
    if op == "spmv":
        return s["A"].spmv(s["x"], s["y"])
    if op == "cg":
        s["A"].cg(s["b"], s["x"], case["iters"])
        return s["x"]
    if op == "pagerank":
        s["x"].fill_(1.0 / s["x"].numel())
        return s["A"].pagerank(DAMPING, case["iters"], s["x"])
    if op == "batched":
        lilac.lilac_spmv_batched(s["handles"], s["xs"], s["ys"])
        return s["y"]
    if op == "bfs":
        return dict(levels=s["A"].bfs(s["source"], s["level"]), level=s["level"])
    if op == "dot":
        lilac.lilac_dot_dev(case["n"], s["a"], s["b"], s["out"])
        return s["out"]
    J = s["J"]
    return lilac.lilac_spmv_jds(s["n"], J["max_len"], J["perm"], J["nzcnt"], J["jd_ptr"],
                                J["col_ind"], J["val"], s["x"], s["y"])


# ------------------------------------------------------------------- the work

def _stencil_nnz(k, points):
    return 7 * k ** 3 - 6 * k * k if points == 7 else (3 * k - 2) ** 3


def _distinct(n, draws):
    """Expected distinct outcomes of `draws` draws among n equal ones."""
    return n * -math.expm1(draws * math.log1p(-1.0 / n)) if n > 1 else 1.0


def _rmat_nnz(scale, edges):
    """Expected distinct edges: cells of the adjacency grouped by how often
    each quadrant was taken."""
    total = 0.0
    for i in range(scale + 1):
        for j in range(scale + 1 - i):
            for k in range(scale + 1 - i - j):
                m = scale - i - j - k
                cells = math.comb(scale, i) * math.comb(scale - i, j) * math.comb(scale - i - j, k)
                p = 0.57 ** i * 0.19 ** (j + k) * 0.05 ** m
                total += cells * -math.expm1(edges * math.log1p(-p))
    return total


def _shape(case):
    """(rows, expected entries) of the case's matrix."""
    kind = case["kind"]
    if kind == "stencil":
        return case["k"] ** 3, _stencil_nnz(case["k"], case["points"])
    if kind == "rmat":
        return 1 << case["scale"], _rmat_nnz(case["scale"], case["edges"])
    n = case["n"]
    if kind == "spd":
        return n, n + 2 * _distinct(n * (n - 1) // 2, n * case["half"])
    lo, hi = (case["per_row"],) * 2 if kind == "uniform" else (case["lo"], case["hi"])
    return n, n * sum(_distinct(n, c) for c in range(lo, hi + 1)) / (hi - lo + 1)


def _product_bytes(n, nnz, vs):
    return nnz * (vs + 4) + (n + 1) * 4 + 2 * n * vs


def work(case):
    op = case["op"]
    vs = 4 if case.get("dtype") == "f32" else 8
    if op == "dot":
        return dict(bytes=2 * case["n"] * vs, flops=2 * case["n"])
    if op == "batched":
        total = entries = 0.0
        for kind, n in _batch_specs(case):
            if kind == "rand":
                rows, nnz = n, n * sum(_distinct(n, c) for c in range(5, 61)) / 56
            else:
                rows, nnz = n ** 3, _stencil_nnz(n, 7 if kind == "st7" else 27)
            total += _product_bytes(rows, nnz, vs)
            entries += nnz
        return dict(bytes=total, flops=2 * entries)
    n, nnz = _shape(case)
    if op == "cg":
        # an iteration: the product, then x, r, p read and written and the
        # product's result read and written
        it = case["iters"]
        return dict(bytes=it * (_product_bytes(n, nnz, 8) + 9 * n * 8), flops=it * (2 * nnz + 12 * n))
    if op == "pagerank":
        return dict(bytes=case["iters"] * _product_bytes(n, nnz, 4), flops=case["iters"] * (2 * nnz + 2 * n))
    if op == "bfs":
        return dict(bytes=nnz * 4 + (n + 1) * 4 + n * 4, flops=nnz)
    if op == "jds":
        return dict(bytes=nnz * 12 + 2 * n * 4 + 2 * n * 8, flops=2 * nnz)
    return dict(bytes=_product_bytes(n, nnz, vs), flops=2 * nnz)


# ------------------------------------------------------------ the same in plain torch

def _plain_product(rp, ci, v):
    rows = rp.numel() - 1
    r = torch.repeat_interleave(torch.arange(rows, device=DEVICE), (rp[1:] - rp[:-1]).to(torch.int64))
    c, v = ci.to(torch.int64), v.to(torch.float64)

    def product(x):
        y = torch.zeros(rows, dtype=torch.float64, device=DEVICE)
        return y.index_add_(0, r, v * x[c])
    return product


def _plain_cg(product, b, iters):
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rho = torch.sum(r * r)
    for _ in range(iters):
        q = product(p)
        pq = torch.sum(p * q)
        if float(rho) == 0.0 or float(pq) == 0.0:
            break
        alpha = rho / pq
        x += alpha * p
        r -= alpha * q
        new = torch.sum(r * r)
        p = r + (new / rho) * p
        rho = new
    return x


def exact(case, seed):
    op, g, dt = case["op"], _gen(seed), _dtype(case)
    if op == "bfs":
        return None   # whole numbers
    if op == "dot":
        a, b = _uniform(case["n"], g, dt), _uniform(case["n"], g, dt)
        return torch.sum(a.to(torch.float64) * b.to(torch.float64))
    if op == "batched":
        mats = [_batch_matrix(m, g, dt) for m in _batch_specs(case)]
        rows, at, x = _batch_vectors(case, g)
        y = torch.zeros(x.numel(), dtype=torch.float64, device=DEVICE)
        for m, a, r in zip(mats, at, rows):
            y[a:a + r] = _plain_product(*m)(x[a:a + r].to(torch.float64))
        return y
    rp, ci, v = _matrix(case, g)
    n = rp.numel() - 1
    product = _plain_product(rp, ci, v)
    if op == "cg":
        return _plain_cg(product, _uniform(n, g, torch.float64), case["iters"])
    if op == "pagerank":
        x = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEVICE)
        for _ in range(case["iters"]):
            x = DAMPING * product(x) + (1.0 - DAMPING) / n
        return x
    y = product(_uniform(n, g, torch.float64 if op == "jds" else dt).to(torch.float64))
    return y.cpu().numpy() if op == "raw" else y
