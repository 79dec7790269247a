"""New values in the column panels, filled in place: bit for bit the products of a
handle created with them, in the lane form (one and more groups of panels, two
blocks to a workgroup), in the scan form, captured graphs and solves included,
both types, again and again."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _rect(rows, cols, lo, hi, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(lo, hi + 1, rows)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return gen.Csr(rows, cols, rp, rng.integers(0, cols, rp[-1]).astype(np.int32),
                   rng.uniform(-1, 1, rp[-1]), f"rect{rows}x{cols}")


MATS = {
    "shared_lines": lambda: _rect(60000, 9000, 1, 100, 1),
    "one_block_panels": lambda: _rect(3000, 200000, 60, 100, 2),
    "groups": lambda: gen.random_rows(100000, 5, 60, seed=3),
    "pairs": lambda: _rect(120000, 120000, 70, 90, 4),
    # few entries to a run: the scan form, 12 bytes an entry against 10 and fillers
    "short_runs": lambda: _rect(400000, 400000, 8, 12, 5),
    "empty_rows": lambda: _rect(50000, 50000, 0, 30, 6),
}


@pytest.mark.parametrize("name", sorted(MATS))
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_updated_equals_new(name, dtype):
    A = MATS[name]().astype(dtype)
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(L.LAYOUT_PANELS)
    assert h.info().layout == L.LAYOUT_PANELS
    bytes0 = h.info().device_bytes
    x = torch.from_numpy(gen.vector(A.cols, 7, dtype=dtype)).to(DEV)
    ys = [torch.empty(A.rows, dtype=x.dtype, device=DEV) for _ in range(3)]
    h.spmv(x, ys[0])
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        h.spmv(x, ys[1])
    for k in range(3):
        v = np.random.default_rng(20 + k).uniform(-1, 1, A.nnz).astype(dtype)
        h.update_values(v if k != 1 else torch.from_numpy(v).to(DEV))
        assert h.info().device_bytes == bytes0
        n = L.Csr(A.row_ptr, A.col_idx, v, cols=A.cols)
        n.set_layout(L.LAYOUT_PANELS)
        for y in ys:
            y.fill_(float("nan"))
        h.spmv(x, ys[0])
        g.replay()
        n.spmv(x, ys[2])
        torch.cuda.synchronize()
        assert torch.equal(ys[0], ys[2]) and torch.equal(ys[1], ys[2])
        L.lilac_spmv_batched([h], [x], [ys[1]])
        torch.cuda.synchronize()
        assert torch.equal(ys[1], ys[2])
        n.destroy()
    h.destroy()


def test_solves_after_new_values():
    A = gen.spd_random(40000, 60, seed=8)
    h = L.Csr.from_gen(A, cols=A.cols)
    assert h.info().layout == L.LAYOUT_PANELS
    b = torch.from_numpy(gen.vector(A.rows, 9)).to(DEV)
    x, want = torch.empty_like(b), torch.empty_like(b)
    h.cg(b, x, 10)
    v = A.vals * 2.0
    h.update_values(v)
    h.cg(b, x, 10)          # the graph captured before
    n = L.Csr(A.row_ptr, A.col_idx, v, cols=A.cols)
    n.cg(b, want, 10)
    torch.cuda.synchronize()
    assert torch.equal(x, want)
    h.destroy()
    n.destroy()
