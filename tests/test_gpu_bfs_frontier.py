"""BFS over frontier bitmaps: graphs with hubs (rows of every length class and
split rows), long chains (many levels in several batches), a frontier that
takes more than one LDS part, isolated vertices, repeated searches; levels bit
for bit against the oracle."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu


def _graph(n, dst, src):
    key = np.unique(dst.astype(np.int64) * n + src)
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rp[1:])
    return gen.Csr(n, n, rp.astype(np.int32), (key % n).astype(np.int32),
                   np.ones(key.size, np.float32), f"graph{n}")


def _two_way(n, a, b):
    return _graph(n, np.concatenate([a, b]), np.concatenate([b, a]))


def _hubs():
    rng = np.random.default_rng(1)
    n = 30000
    a = [rng.integers(0, n, 20000)]
    b = [rng.integers(0, n, 20000)]
    for i, k in enumerate((3, 7, 40, 100, 200, 700, 3000, 9000, 20000)):
        a.append(np.full(k, 11 * i))
        b.append(rng.choice(n, k, replace=False))
    return _two_way(n, np.concatenate(a), np.concatenate(b))


GRAPHS = {
    "hubs": (_hubs, 17),
    "chain_7": (lambda: _two_way(8, np.arange(7), np.arange(1, 8)), 0),
    "chain_200": (lambda: _two_way(201, np.arange(200), np.arange(1, 201)), 0),
    "isolated": (lambda: _graph(1000, np.array([5]), np.array([6])), 6),
    "two_parts": (lambda: _two_way(1400000, np.arange(0, 1399999, 7),
                                   (np.arange(0, 1399999, 7) * 5 + 3) % 1400000), 3),
    "rmat": (lambda: gen.rmat_pagerank(15, 1 << 18), 12),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_levels(name):
    make, source = GRAPHS[name]
    A = make()
    if name == "rmat":
        source = int(A.col_idx[A.nnz // 2])
    h = L.Csr.from_gen(A, cols=A.cols)
    ref = oracle.bfs_levels(A.row_ptr, A.col_idx, source)
    ref = ref[0] if isinstance(ref, tuple) else ref
    level = torch.empty(A.rows, dtype=torch.int32, device="cuda")
    for _ in range(2):
        n = h.bfs(source, level)
        assert np.array_equal(level.cpu().numpy(), ref)
        assert n == ref.max() + 1
    h.destroy()
