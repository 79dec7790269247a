"""BFS with as many vertices as the frontier's bits in LDS hold (160 KB), one more
and twice as many (bits in device memory), levels bit for bit against the oracle;
rows of every class, many levels."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1310720, 1310721, 2621500])
def test_levels_at_the_lds_edge(n):
    rng = np.random.default_rng(n)
    # a chain through every 30,000th vertex, bushes on it, hubs of every class
    chain = np.arange(0, n - 1, 30000)
    a = [chain[:-1], rng.integers(0, n, 3 * n // 4)]
    b = [chain[1:], np.zeros(3 * n // 4, np.int64)]
    b[1] = np.minimum(a[1] + rng.integers(1, 2000, a[1].size), n - 1)
    for i, k in enumerate((5, 33, 129, 513, 2000, 9000)):
        a.append(np.full(k, n - 1 - 7 * i))
        b.append(rng.choice(n, k, replace=False))
    a, b = np.concatenate(a), np.concatenate(b)
    key = np.unique(np.concatenate([a * n + b, b * n + a]))
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rp[1:])
    A = gen.Csr(n, n, rp.astype(np.int32), (key % n).astype(np.int32),
                np.ones(key.size, np.float32), f"edge{n}")
    h = L.Csr.from_gen(A, cols=n)
    ref = oracle.bfs_levels(A.row_ptr, A.col_idx, 0)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert ref.max() > 20
    level = torch.empty(n, dtype=torch.int32, device="cuda")
    for _ in range(2):
        assert h.bfs(0, level) == ref.max() + 1
        assert np.array_equal(level.cpu().numpy(), ref)
    h.destroy()
