"""Hot-column layout of matrices most of whose rows are empty (more spans of
empty rows than workgroups, rows with entries first or apart), against the
oracle."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("apart", [False, True])
@pytest.mark.parametrize("dtype", (np.float64, np.float32))
def test_mostly_empty(apart, dtype):
    rows, cols, filled, each = 6_500_000, 90_000, 60_000, 40
    rng = np.random.default_rng(5)
    lens = np.zeros(rows, dtype=np.int64)
    lens[np.sort(rng.choice(rows, filled, replace=False)) if apart else np.arange(filled)] = each
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = (cols * rng.random(rp[-1]) ** 3).astype(np.int32)
    A = gen.Csr(rows, cols, rp.astype(np.int32), c, rng.uniform(-1, 1, rp[-1]), "sparse").astype(dtype)
    h = L.Csr.from_gen(A, cols=cols)
    h.set_layout(L.LAYOUT_HOT)
    x = gen.vector(cols, 6, dtype=dtype)
    xd = torch.from_numpy(x).cuda()
    y = torch.full((rows,), np.nan, dtype=xd.dtype, device="cuda")
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64 if dtype == np.float64 else TOL_F32)
    h.destroy()
