"""Raw calls around the size up to which vectors go through pinned memory, for
layouts that store to it directly and the row-class tiles, both types; one
vector on the device and the other not; sizes that are not whole 16 bytes."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5, 255, 3001, 32767, 32768, 32769, 65537])
@pytest.mark.parametrize("kind", ["diagonals", "random"])
def test_sizes(n, kind):
    rng = np.random.default_rng(n)
    if kind == "diagonals":
        cols = np.clip(np.arange(n)[:, None] + np.array([-3, 0, 2]), 0, n - 1)
    else:
        cols = rng.integers(0, n, (n, 3))
    rp = (np.arange(n + 1) * 3).astype(np.int32)
    A = gen.Csr(n, n, rp, cols.reshape(-1).astype(np.int32), rng.uniform(-1, 1, 3 * n), kind)
    for dtype, call, tol in ((np.float64, L.lilac_spmv_csr, TOL_F64),
                             (np.float32, L.lilac_spmv_csr_f32, TOL_F32)):
        B = A.astype(dtype)
        for a in (B.row_ptr, B.col_idx, B.vals):
            L.lilac_invalidate(a)
        for k in range(2):
            x = gen.vector(n, 50 + k, dtype=dtype)
            y = np.full(n + 1, 7.0, dtype=dtype)
            call(n, B.row_ptr, B.col_idx, B.vals, x, y)
            assert y[n] == 7.0   # nothing past the rows
            check_spmv(B, x, y[:n], tol)
            yd = torch.empty(n, dtype=torch.from_numpy(x).dtype, device="cuda")
            call(n, B.row_ptr, B.col_idx, B.vals, x, yd)
            assert np.array_equal(yd.cpu().numpy(), y[:n])
            z = np.empty(n, dtype=dtype)
            call(n, B.row_ptr, B.col_idx, B.vals, torch.from_numpy(x).cuda(), z)
            assert np.array_equal(z, y[:n])
    L.lilac_release_all()
