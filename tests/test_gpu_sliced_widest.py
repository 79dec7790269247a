"""Stencils with one longer row: the sliced form of the band layout (10 bytes an
entry) is taken only up to a bound on that row (one lane adds it up), the scan
form (which keeps the values in place: 4 more bytes an entry) past it; the device
bytes tell which, results against the oracle, grouped equal to single."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu


def _with_long_row(k, points, width):
    A = gen.stencil(k, points)
    i = A.rows // 2
    a, z = int(A.row_ptr[i]), int(A.row_ptr[i + 1])
    c0 = i - width // 2
    rng = np.random.default_rng(width)
    col = np.concatenate([A.col_idx[:a], np.arange(c0, c0 + width, dtype=np.int32), A.col_idx[z:]])
    vals = np.concatenate([A.vals[:a], rng.uniform(-1, 1, width), A.vals[z:]])
    rp = A.row_ptr.copy()
    rp[i + 1:] += width - (z - a)
    return gen.Csr(A.rows, A.cols, rp, col, vals, f"st{k}p{points}w{width}")


# 64^3 rows are 4096 slices, a line of the grid each: 27 points 3 (3 * 64 - 2)^2 =
# 108300 columns of 64, a 1024th of them 105; 7 points fewer (the floor of 64
# holds); 40^3 rows are 1000 slices (the floor of 32)
@pytest.mark.parametrize("k,points,width,sliced", [
    (64, 27, 105, True), (64, 27, 106, False), (64, 27, 30000, False),
    (64, 7, 64, True), (64, 7, 65, False),
    (40, 27, 32, True), (40, 27, 33, False)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_widest_row(k, points, width, sliced, dtype):
    A = _with_long_row(k, points, width).astype(dtype)
    h = L.Csr.from_gen(A, cols=A.cols)
    inf = h.info()
    assert inf.layout == L.LAYOUT_BAND
    vs = np.dtype(dtype).itemsize
    copy = inf.device_bytes - A.nnz * (vs + 4) - A.rows * 8
    assert (copy > A.nnz * (vs + 2)) == sliced
    x = gen.vector(A.cols, 3, dtype=dtype)
    xd = torch.from_numpy(x).cuda()
    y = torch.full((A.rows,), np.nan, dtype=xd.dtype, device="cuda")
    y2 = y.clone()
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64 if dtype == np.float64 else TOL_F32)
    L.lilac_spmv_batched([h], [xd], [y2])
    assert torch.equal(y, y2)
    h.destroy()
