"""Requests served equal single calls bit for bit whatever layout the matrix gets:
hub matrices over renamed hot columns, groups of panels, lane forms larger than
the scan form, slices; the plain path's CG equals lilac_cg."""
import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L
from tests.helpers import TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _hubs(rows, cols, per, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 2 * per, rows)
    lens[9] = 3000
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = rng.permutation(cols)[(cols * rng.random(rp[-1]) ** 4).astype(np.int64)]
    return gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                   rng.uniform(-1, 1, rp[-1]), f"hubs{rows}x{cols}")


MATS = {"hubs": lambda: _hubs(260000, 300000, 15, 1),
        # many entries a row: little room but the copy's own in the bound
        "heavy_hubs": lambda: _hubs(60000, 900000, 90, 2),
        "groups": lambda: gen.random_rows(120000, 5, 60, seed=3),
        "lanes": lambda: gen.random_rows(400000, 5, 30, seed=4),
        "slices": lambda: gen.stencil(60, 27)}


@pytest.mark.parametrize("fifo", [False, True])
@pytest.mark.parametrize("name", sorted(MATS))
def test_served_product_equals_single(name, fifo):
    A = MATS[name]()
    h = L.Csr.from_gen(A, cols=A.cols)
    if "hubs" in name:
        assert h.info().layout == L.LAYOUT_HOT
    x = gen.vector(A.cols, 5)
    xd = torch.from_numpy(x).to(DEV)
    want = torch.empty(A.rows, dtype=torch.float64, device=DEV)
    h.spmv(xd, want)
    torch.cuda.synchronize()
    h.destroy()
    S = L.Server(fifo=fifo)
    mid = S.add_matrix(A)
    got = torch.full_like(want, float("nan"))
    torch.cuda.synchronize()
    S.wait(S.submit(L.REQ_SPMV, mid, xd, got))
    torch.cuda.synchronize()
    assert S.stats()["failed"] == 0
    S.destroy()
    check_spmv(A, x, want.cpu().numpy(), TOL_F64)
    assert torch.equal(got, want)


@pytest.mark.parametrize("name", ["fused", "slices", "groups"])
def test_plain_path_solve_equals_lilac_cg(name):
    A = {"fused": lambda: gen.stencil(26, 7), "slices": lambda: gen.stencil(30, 27),
         "groups": lambda: gen.spd_random(60000, 25, seed=6)}[name]()
    h = L.Csr.from_gen(A, cols=A.cols)
    b = torch.from_numpy(gen.vector(A.rows, 7)).to(DEV)
    want, got = torch.empty_like(b), torch.full_like(b, float("nan"))
    h.cg(b, want, 20)
    torch.cuda.synchronize()
    h.destroy()
    S = L.Server(fifo=True)
    mid = S.add_matrix(A)
    S.wait(S.submit(L.REQ_CG, mid, b, got, iters=20))
    torch.cuda.synchronize()
    S.destroy()
    assert torch.equal(got, want)
