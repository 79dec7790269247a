"""Hot-column layout of matrices of few non-empty rows: blocks of the least
entries, blocks grown until no workgroup has two, rows that fill half of the
blocks and a little more, single huge rows; against the oracle."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu


def _graph(rows, cols, filled, nnz, seed):
    """`filled` non-empty rows of power-law lengths, power-law columns."""
    rng = np.random.default_rng(seed)
    own = np.sort(rng.choice(rows, filled, replace=False))
    share = (np.arange(filled) + 1.0) ** -0.7
    lens = np.zeros(rows, dtype=np.int64)
    lens[own] = 1 + (nnz * share / share.sum()).astype(np.int64)
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = (cols * rng.random(rp[-1]) ** 3).astype(np.int64)
    return gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                   rng.uniform(-1, 1, rp[-1]), f"graph{rows}x{cols}")


@pytest.mark.parametrize("rows,cols,filled,nnz", [
    (70000, 65000, 40, 300),                # one block
    (65536, 65536, 35000, 600_000),         # 4096 entries a block
    (262144, 100000, 150_000, 2_500_000),   # grown until one to a workgroup
    (300000, 90000, 196_608, 1_100_000),    # rows of half the blocks
    (300000, 90000, 196_609, 1_100_000),    # and one more
    (50000, 80000, 3, 900_000),             # three rows
])
@pytest.mark.parametrize("dtype", (np.float64, np.float32))
def test_few_blocks(rows, cols, filled, nnz, dtype):
    A = _graph(rows, cols, filled, nnz, rows + filled).astype(dtype)
    h = L.Csr.from_gen(A, cols=cols)
    h.set_layout(L.LAYOUT_HOT)
    assert h.info().layout == L.LAYOUT_HOT
    x = gen.vector(cols, 41, dtype=dtype)
    xd = torch.from_numpy(x).cuda()
    y, z = [torch.full((rows,), np.nan, dtype=xd.dtype, device="cuda") for _ in range(2)]
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64 if dtype == np.float64 else TOL_F32)
    h.spmv(xd, z)
    assert torch.equal(y, z)
    h.destroy()
