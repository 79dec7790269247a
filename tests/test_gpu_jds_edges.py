"""JDS product on device arrays: diagonals around the group that is loaded
together, bitwise against the oracle; arrays at fault are refused with y left
as it was."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _dev(J):
    return {k: torch.from_numpy(np.ascontiguousarray(getattr(J, k))).to(DEV)
            for k in ("perm", "nzcnt", "jd_ptr", "jd_col", "jd_val")}


def _call(J, d, x, y):
    L.lilac_spmv_jds(J.rows, J.max_len, d["perm"], d["nzcnt"],
                     d["jd_ptr"], d["jd_col"], d["jd_val"], x, y)


@pytest.mark.parametrize("rows", [1, 64, 257, 3000])
@pytest.mark.parametrize("max_len", [1, 7, 8, 9, 16, 23])
def test_diagonal_groups(rows, max_len):
    J = gen.random_jds(rows, 500, max_len, seed=rows + max_len)
    if J.max_len == 0:
        pytest.skip("all rows empty")
    x = gen.vector(500, 3)
    ref = oracle.spmv_jds(dict(perm=J.perm, nzcnt=J.nzcnt, jd_ptr=J.jd_ptr, col_ind=J.jd_col,
                               val=J.jd_val, max_len=J.max_len), x)
    d = _dev(J)
    y = torch.full((rows,), np.nan, dtype=torch.float64, device=DEV)
    for _ in range(2):   # the second call finds the kept permutation buffer
        _call(J, d, torch.from_numpy(x).to(DEV), y)
        assert np.array_equal(y.cpu().numpy(), ref)


def test_faults_leave_y():
    J = gen.random_jds(1000, 300, 12, seed=5)
    x = torch.from_numpy(gen.vector(300, 4)).to(DEV)
    y = torch.full((1000,), 7.0, dtype=torch.float64, device=DEV)
    d = _dev(J)
    d["jd_col"][-1] = -1
    with pytest.raises(L.LilacError) as e:
        _call(J, d, x, y)
    assert e.value.code == -2 and bool((y == 7.0).all())
    d = _dev(J)
    d["jd_ptr"][-1] = -5
    with pytest.raises(L.LilacError) as e:
        _call(J, d, x, y)
    assert e.value.code == -1 and bool((y == 7.0).all())
    # a row whose position is not one is not stored
    d = _dev(J)
    d["perm"][3] = -1
    _call(J, d, x, y)
    assert y[3].item() == 7.0
