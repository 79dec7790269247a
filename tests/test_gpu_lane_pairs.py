"""Lane form of the column panels with several row blocks to a workgroup of a
grouped launch: block counts that do not divide, one, two and four together,
one and several panels, with and without groups of panels, both types; grouped
equal to single bit for bit, whole numbers exactly; CG on a server, whose
grouped products also write the partials of a dot."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L
from tests.helpers import TOL_F32, TOL_F64, check_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda"

# rows, entries per row: blocks weigh one copy of x (about 8 n / 12 len rows)
SHAPES = [(5000, 30), (5100, 33), (9000, 20), (12000, 70), (30000, 12), (31000, 11), (40000, 24),
          (60000, 12), (75000, 30), (150000, 14)]


def _mat(n, length, dtype):
    rng = np.random.default_rng(n)
    lens = rng.integers(length // 2, length + length // 2, n)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    c = rng.integers(0, n, rp[-1]).astype(np.int32)
    return gen.Csr(n, n, rp, c, rng.uniform(-1, 1, rp[-1]), f"rows{n}x{length}").astype(dtype)


@pytest.mark.parametrize("dtype", (np.float64, np.float32))
def test_grouped_equals_single(dtype):
    tol = TOL_F64 if dtype == np.float64 else TOL_F32
    mats = [_mat(n, length, dtype) for n, length in SHAPES]
    hs = [L.Csr.from_gen(A, cols=A.cols) for A in mats]
    for h in hs:
        h.set_layout(L.LAYOUT_PANELS)
    xs = [gen.vector(A.cols, k, dtype=dtype) for k, A in enumerate(mats)]
    xd = [torch.from_numpy(x).to(DEV) for x in xs]
    single, many = [[torch.full((A.rows + 1,), np.nan, dtype=v.dtype, device=DEV)
                     for A, v in zip(mats, xd)] for _ in range(2)]
    for h, v, y in zip(hs, xd, single):
        h.spmv(v, y[:-1])
    # few blocks (one to a workgroup), then enough of them for four
    for copies in (1, 2, 8):
        ys = [[torch.full_like(y, np.nan) for y in many] for _ in range(copies)]
        L.lilac_spmv_batched(hs * copies, xd * copies, [y[:-1] for some in ys for y in some])
        torch.cuda.synchronize()
        for some in ys:
            assert all(torch.equal(y[:-1], z[:-1]) for y, z in zip(single, some))
            assert all(bool(torch.isnan(z[-1])) for z in some)
    L.lilac_spmv_batched(hs, xd, [y[:-1] for y in many])
    torch.cuda.synchronize()
    for A, x, y, z in zip(mats, xs, single, many):
        check_spmv(A, x, y[:-1].cpu().numpy(), tol)
        assert torch.equal(y[:-1], z[:-1])
        assert bool(torch.isnan(z[-1]))
    for A, h, y in zip(mats, hs, many):
        h.update_values(gen.int_vector(A.nnz, 5).astype(dtype))
    xi = [gen.int_vector(A.cols, 6).astype(dtype) for A in mats]
    ys = [[torch.empty_like(y) for y in many] for _ in range(8)]
    L.lilac_spmv_batched(hs * 8, [torch.from_numpy(x).to(DEV) for x in xi] * 8,
                         [y[:-1] for some in ys for y in some])
    many = ys[7]
    for A, x, y in zip(mats, xi, many):
        want = oracle.spmv_csr(A.row_ptr, A.col_idx, gen.int_vector(A.nnz, 5), x.astype(np.float64))
        assert np.array_equal(y[:-1].cpu().numpy().astype(np.float64), want)
    for h in hs:
        h.destroy()


def test_server_cg():
    """Grouped products with dot partials: alone and together the same bits."""
    mats = [gen.spd_random(5000, 20, seed=1), gen.spd_random(12000, 12, seed=2),
            gen.spd_random(30000, 6, seed=3), gen.spd_random(50000, 40, seed=4)]
    S = L.Server()
    ids = [S.add_matrix(A) for A in mats]
    bs = [gen.vector(A.rows, 30 + k) for k, A in enumerate(mats)]
    bd = [torch.from_numpy(b).to(DEV) for b in bs]

    def run(together, copies=1):
        outs = [torch.full_like(b, np.nan) for b in bd * copies]
        torch.cuda.synchronize()
        tickets = []
        for mid, b, o in zip(ids * copies, bd * copies, outs):
            tickets.append(S.submit(L.REQ_CG, mid, b, o, iters=12))
            if not together:
                S.wait(tickets[-1])
        for t in tickets:
            S.wait(t)
        torch.cuda.synchronize()
        return outs

    alone, mixed, many = run(False), run(True), run(True, 12)
    assert all(torch.equal(a, m) for a, m in zip(alone * 12, many))
    for A, b, a, m in zip(mats, bs, alone, mixed):
        assert torch.equal(a, m)
        ref, _, _ = oracle.cg(A.row_ptr, A.col_idx, A.vals, b, 12)
        assert np.max(np.abs(a.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref))
    S.destroy()
