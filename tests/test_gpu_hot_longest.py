"""Hub matrices with one very long row: the hot-column layout over renamed
columns is chosen by itself only while no row outweighs three workgroups' shares
of the entries (a row is never cut there); both sides of the rule against the
oracle."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("share,layout", [(2.9, L.LAYOUT_HOT), (3.1, L.LAYOUT_ROWS),
                                          (52.0, L.LAYOUT_ROWS)])
def test_longest_row(dtype, share, layout):
    rows, cols = 200000, 250000
    rng = np.random.default_rng(11)
    lens = rng.integers(1, 40, rows)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # longest = share * nnz / cus with the row itself among the nnz
    lens[4321] = int(share * lens.sum() / (cus - share))
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = rng.permutation(cols)[(cols * rng.random(rp[-1]) ** 4).astype(np.int64)]
    A = gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                rng.uniform(-1, 1, rp[-1]), "longest").astype(dtype)
    assert A.nnz >= 3000000
    h = L.Csr.from_gen(A, cols=cols)
    assert h.info().layout == layout
    x = gen.vector(cols, 12, dtype=dtype)
    xd = torch.from_numpy(x).cuda()
    y = torch.full((rows,), np.nan, dtype=xd.dtype, device="cuda")
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64 if dtype == np.float64 else TOL_F32)
    h.destroy()
