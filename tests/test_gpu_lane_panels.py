"""Lane form of the column-panel layout: run lengths around the 64 equal
pieces and the pairs of columns, rows with gaps between panels (fillers),
rows that span many lanes, last blocks of few rows, both types, several
panels, against the oracle; grouped equal to single; fillers and padding
never multiply an infinity."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rows(lens, cols, seed, clustered=False):
    """Row i: lens[i] random columns (repeats allowed); clustered: a third of
    the rows has columns of the first half only, a third of the second."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    r = np.repeat(np.arange(lens.size), lens)
    lo, hi = np.zeros(r.size), np.full(r.size, float(cols))
    if clustered:
        hi[r % 3 == 0] = cols / 2
        lo[r % 3 == 1] = cols / 2
    c = np.minimum((lo + rng.random(r.size) * (hi - lo)).astype(np.int64), cols - 1)
    return gen.Csr(lens.size, cols, rp, c.astype(np.int32), rng.uniform(-1, 1, r.size),
                   f"rows{lens.size}x{cols}")


def _mats():
    rng = np.random.default_rng(1)
    yield "one_row", _rows([5000], 3000, 2)
    yield "even_runs", _rows(np.full(512, 64), 4000, 3)
    yield "odd_runs", _rows(np.full(4096, 17), 15000, 4)
    yield "short_last_block", _rows(np.full(1025, 90), 30000, 5)
    yield "gaps", _rows(rng.integers(20, 60, 6000), 60000, 6, clustered=True)
    yield "empty_rows", _rows(np.where(rng.random(5000) < 0.2, 0, 70), 30000, 7)
    yield "long_rows", _rows(np.where(np.arange(3000) % 100 == 0, 2500, 30), 45000, 8)
    yield "many_blocks", _rows(rng.integers(100, 300, 40000), 40000, 9)


MATS = dict(_mats())


def _handle(A):
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(L.LAYOUT_PANELS)
    assert h.info().layout == L.LAYOUT_PANELS
    return h


@pytest.mark.parametrize("name", sorted(MATS))
def test_runs(name):
    A = MATS[name]
    x = gen.vector(A.cols, 21)
    xd = torch.from_numpy(x).to(DEV)
    h = _handle(A)
    y = torch.full((A.rows,), np.nan, dtype=torch.float64, device=DEV)
    h.spmv(xd, y)
    check_spmv(A, x, y.cpu().numpy(), TOL_F64)
    y2 = torch.full_like(y, np.nan)
    L.lilac_spmv_batched([h, h], [xd, xd], [torch.empty_like(y), y2])
    assert torch.equal(y, y2)
    w, out = gen.vector(A.rows, 22), torch.empty(1, dtype=torch.float64, device=DEV)
    h.spmv_dot(xd, y2, torch.from_numpy(w).to(DEV), out)
    assert torch.equal(y, y2)
    yh = y.cpu().numpy()
    assert abs(out.item() - oracle.dot(w, yh)) <= TOL_F64 * oracle.dot_abs(w, yh)
    # x that is not 16-byte aligned; whole numbers exactly
    B = gen.Csr(A.rows, A.cols, A.row_ptr, A.col_idx, gen.int_vector(A.nnz, 23), "int")
    xi = gen.int_vector(A.cols, 24)
    off = torch.empty(A.cols + 1, dtype=torch.float64, device=DEV)
    off[1:] = torch.from_numpy(xi).to(DEV)
    h.update_values(B.vals)
    h.spmv(off[1:], y)
    assert np.array_equal(y.cpu().numpy(), oracle.spmv_csr(B.row_ptr, B.col_idx, B.vals, xi))
    h.destroy()
    C = A.astype(np.float32)
    x32 = gen.vector(A.cols, 25, dtype=np.float32)
    h = _handle(C)
    y = torch.full((A.rows,), np.nan, dtype=torch.float32, device=DEV)
    h.spmv(torch.from_numpy(x32).to(DEV), y)
    check_spmv(C, x32, y.cpu().numpy(), TOL_F32)
    h.destroy()


@pytest.mark.parametrize("name", ["gaps", "empty_rows", "odd_runs"])
def test_fillers_keep_infinities_apart(name):
    """Every x infinite, values of one sign: rows are +Inf, empty ones 0."""
    A = MATS[name]
    B = gen.Csr(A.rows, A.cols, A.row_ptr, A.col_idx, np.abs(A.vals) + 0.5, "pos")
    h = _handle(B)
    x = torch.full((A.cols,), np.inf, dtype=torch.float64, device=DEV)
    y = torch.empty(A.rows, dtype=torch.float64, device=DEV)
    h.spmv(x, y)
    want = np.where(np.diff(A.row_ptr) > 0, np.inf, 0.0)
    assert np.array_equal(y.cpu().numpy(), want)
    h.destroy()
