"""New values while products and solves enqueued before are still to run: those
use the old values, bit for bit, in every layout that keeps a copy of them
(hot columns, sliced and scan band, column panels) and in the row-class tiles."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _mats():
    return {
        "hot": (gen.random_rows(200000, 5, 60, seed=31), L.LAYOUT_HOT),
        "sliced": (gen.stencil(60, 27), L.LAYOUT_BAND),
        "band": (gen.ragged(60000, 3000, seed=32, max_len=60), L.LAYOUT_BAND),
        "panels": (gen.random_rows(100000, 5, 60, seed=33), L.LAYOUT_PANELS),
        "rows": (gen.random_rows(200000, 5, 60, seed=34), L.LAYOUT_ROWS),
    }


@pytest.mark.parametrize("name", ["hot", "sliced", "band", "panels", "rows"])
@pytest.mark.parametrize("device_vals", [False, True])
def test_queued_products_use_the_old_values(name, device_vals):
    A, layout = _mats()[name]
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(layout)
    x = torch.from_numpy(gen.vector(A.cols, 1)).to(DEV)
    want = torch.empty(A.rows, dtype=torch.float64, device=DEV)
    h.spmv(x, want)
    ys = [torch.full_like(want, float("nan")) for _ in range(60)]
    other = A.vals * 3.0 + 1.0
    vals = torch.from_numpy(other).to(DEV) if device_vals else other
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for y in ys:
        h.spmv(x, y, stream=s)
    h.update_values(vals)
    after = torch.empty_like(want)
    h.spmv(x, after)
    torch.cuda.synchronize()
    for y in ys:
        assert torch.equal(y, want)
    g = L.Csr(A.row_ptr, A.col_idx, other, cols=A.cols)
    g.set_layout(layout)
    h.spmv(x, want)
    g.spmv(x, ys[0])
    assert torch.equal(after, want) and torch.equal(after, ys[0])
    h.destroy()
    g.destroy()


@pytest.mark.parametrize("layout", [L.LAYOUT_HOT, L.LAYOUT_BAND])
def test_queued_solve_uses_the_old_values(layout):
    A = gen.stencil(70, 27)
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(layout)
    b = torch.from_numpy(gen.vector(A.rows, 2)).to(DEV)
    want, got = torch.empty_like(b), torch.empty_like(b)
    h.cg(b, want, 60)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    h.cg(b, got, 60, stream=s)
    h.update_values(A.vals * np.where(A.vals > 0, 2.0, 1.0))
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    h.destroy()
