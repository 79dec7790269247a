"""Hot-column layout over renamed columns, chosen by itself for large matrices
with scattered hub columns and rows too long for the column panels: against the
oracle row by row, both types; the same bits in a batch, after a replayed
capture and where the stream has no working memory; new values; blocks around
the parts in which they are cut; the fused dot."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"
PER_THREAD = 2   # hipStreamPerThread: no working memory of its own


def _hubs(rows, cols, seed):
    """Power-law columns under a random renaming, a third of the rows empty,
    some rows of thousands of entries (repeats allowed)."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 60, rows)
    lens[rng.random(rows) < 0.33] = 0
    lens[rng.choice(rows, 20, replace=False)] = rng.integers(1025, 20000, 20)
    lens[-1] = 0
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = rng.permutation(cols)[(cols * rng.random(rp[-1]) ** 4).astype(np.int64)]
    return gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                   rng.uniform(-1, 1, rp[-1]), f"hubs{rows}x{cols}")


@pytest.mark.parametrize("rows,cols", [(170001, 300000), (420000, 170000)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_renamed_columns(rows, cols, dtype):
    A = _hubs(rows, cols, rows).astype(dtype)
    assert A.nnz >= 3000000
    tol = TOL_F64 if dtype == np.float64 else TOL_F32
    h = L.Csr.from_gen(A, cols=cols)
    assert h.info().layout == L.LAYOUT_HOT
    x = gen.vector(cols, 31, dtype=dtype)
    xd = torch.from_numpy(x).to(DEV)
    y = torch.full((rows,), np.nan, dtype=xd.dtype, device=DEV)
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), tol)
    other = torch.full_like(y, np.nan)
    h.spmv(xd, other, stream=PER_THREAD)
    torch.cuda.synchronize()
    assert torch.equal(y, other)
    other.fill_(np.nan)
    L.lilac_spmv_batched([h], [xd], [other])
    assert torch.equal(y, other)
    # captured: replays with eager work between them
    g, cx, cy = torch.cuda.CUDAGraph(), xd.clone(), torch.empty_like(y)
    with torch.cuda.graph(g):
        h.spmv(cx, cy)
    for k in range(3):
        x2 = torch.from_numpy(gen.vector(cols, 40 + k, dtype=dtype)).to(DEV)
        cx.copy_(x2)
        g.replay()
        h.spmv(x2, other)
        assert torch.equal(cy, other)
    if dtype == np.float64:
        w, out = gen.vector(rows, 32), torch.empty(1, dtype=torch.float64, device=DEV)
        h.spmv_dot(xd, other, torch.from_numpy(w).to(DEV), out)
        assert torch.equal(y, other)
        yh = y.cpu().numpy()
        assert abs(out.item() - oracle.dot(w, yh)) <= TOL_F64 * oracle.dot_abs(w, yh)
    # new values, whole numbers: exact in either type (sums below 2^24)
    B = gen.Csr(rows, cols, A.row_ptr, A.col_idx, gen.int_vector(A.nnz, 33, dtype=dtype), "int")
    xi = gen.int_vector(cols, 34, dtype=dtype)
    h.update_values(B.vals)
    h.spmv(torch.from_numpy(xi).to(DEV), y)
    ref = oracle.spmv_csr(B.row_ptr, B.col_idx, B.vals, xi)
    assert np.array_equal(y.cpu().numpy().astype(np.float64), ref)
    h.destroy()
