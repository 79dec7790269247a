"""Hot-column layout over renamed columns where x may not be copied into its
order (a captured graph): the bits of the eager product, for columns that all fit
the LDS, columns just past that and many more, both types; new values reach a
graph captured before."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype,cols,skew", [(np.float64, 17281, 2), (np.float64, 90001, 2),
                                             (np.float32, 34561, 2), (np.float32, 500003, 4)])
def test_captured_equals_eager(dtype, cols, skew):
    rows = 190003
    rng = np.random.default_rng(cols)
    # scattered enough for the rule of lines (0.3 a non-zero) on few columns
    lens = rng.integers(10, 25, rows)
    lens[1234] = 2000
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = rng.permutation(cols)[(cols * rng.random(rp[-1]) ** skew).astype(np.int64)]
    A = gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                rng.uniform(-1, 1, rp[-1]), "direct").astype(dtype)
    h = L.Csr.from_gen(A, cols=cols)
    assert h.info().layout == L.LAYOUT_HOT
    x = gen.vector(cols, 3, dtype=dtype)
    xd = torch.from_numpy(x).to(DEV)
    y = torch.full((rows,), np.nan, dtype=xd.dtype, device=DEV)
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64 if dtype == np.float64 else TOL_F32)
    cx, cy, g = xd.clone(), torch.full_like(y, np.nan), torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        h.spmv(cx, cy)
    for k in range(3):
        if k == 2:
            h.update_values(A.vals[::-1].copy())
        x2 = torch.from_numpy(gen.vector(cols, 10 + k, dtype=dtype)).to(DEV)
        cx.copy_(x2)
        g.replay()
        h.spmv(x2, y)
        torch.cuda.synchronize()
        assert torch.equal(cy, y)
    h.destroy()
