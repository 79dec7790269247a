"""Sliced form of the band layout (rows of nearly one length, 64 to a slice):
slice widths around the groups of four, pair and single column, row counts
around the slice, ragged rows inside the padding bound, empty rows, both
types, against the oracle; grouped equal to single; padding never multiplies
an infinity."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _near(rows, cols, lens, seed):
    """Row i: lens[i] columns drawn near the diagonal (repeats allowed)."""
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    r = np.repeat(np.arange(rows), lens)
    c = np.clip(r * cols // max(rows, 1) + rng.integers(-200, 201, r.size), 0, cols - 1)
    return gen.Csr(rows, cols, rp, c.astype(np.int32), rng.uniform(-1, 1, r.size),
                   f"near{rows}w{int(lens.max(initial=0))}")


def _handle(A):
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(L.LAYOUT_BAND)
    assert h.info().layout == L.LAYOUT_BAND
    return h


def _lens(rows, width, short, seed):
    lens = np.full(rows, width)
    if short:   # one row in sixteen shorter, one of them empty
        pick = np.random.default_rng(seed).choice(rows, max(1, rows // 16), replace=False)
        lens[pick] = np.maximum(0, width - 1 - (np.arange(pick.size) % 3))
        lens[pick[0]] = 0
    return lens


@pytest.mark.parametrize("rows", [1, 63, 64, 65, 255, 4097])
@pytest.mark.parametrize("width", [1, 2, 3, 4, 5, 7, 8, 11, 16, 27, 32, 33])
def test_widths_and_row_counts(rows, width):
    A = _near(rows, max(rows, 40), _lens(rows, width, rows > 64, width), rows * 100 + width)
    x = gen.vector(A.cols, 7)
    h = _handle(A)
    y = torch.full((rows,), np.nan, dtype=torch.float64, device=DEV)
    h.spmv(torch.from_numpy(x).to(DEV), y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64)
    y2 = torch.full((rows,), np.nan, dtype=torch.float64, device=DEV)
    L.lilac_spmv_batched([h, h], [torch.from_numpy(x).to(DEV)] * 2, [y2, torch.empty_like(y2)])
    assert torch.equal(y, y2)
    # new values reach the sliced copy
    B = gen.Csr(A.rows, A.cols, A.row_ptr, A.col_idx, gen.int_vector(A.nnz, 9), "int")
    xi = gen.int_vector(A.cols, 10)
    h.update_values(B.vals)
    h.spmv(torch.from_numpy(xi).to(DEV), y)
    import oracle
    assert np.array_equal(y.cpu().numpy(), oracle.spmv_csr(B.row_ptr, B.col_idx, B.vals, xi))
    h.destroy()
    C = A.astype(np.float32)
    x32 = gen.vector(A.cols, 8, dtype=np.float32)
    h = _handle(C)
    y = torch.full((rows,), np.nan, dtype=torch.float32, device=DEV)
    h.spmv(torch.from_numpy(x32).to(DEV), y)
    check_spmv(C, x32, y.cpu().numpy(), TOL_F32)
    h.destroy()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_padding_keeps_infinities_apart(dtype):
    """Every entry of x is infinite: a row is infinite of one sign if its
    values have one sign, NaN only if they have both, 0 if it is empty."""
    rows, width = 1000, 13
    A = _near(rows, rows, _lens(rows, width, True, 3), 5)
    A.vals = np.where(np.arange(A.nnz) % 7 == 0, -1.0, 1.0).astype(dtype)
    h = _handle(A)
    x = torch.full((rows,), np.inf, dtype=torch.float64 if dtype == np.float64 else torch.float32,
                   device=DEV)
    y = torch.zeros_like(x)
    h.spmv(x, y)
    want = np.zeros(rows)
    for i in range(rows):
        v = A.vals[A.row_ptr[i]:A.row_ptr[i + 1]]
        if v.size:
            want[i] = np.inf if (v > 0).all() else -np.inf if (v < 0).all() else np.nan
    np.testing.assert_array_equal(y.cpu().numpy().astype(np.float64), want)
    h.destroy()
