"""CG with one kernel per iteration (small sliced band matrices of short rows):
against the oracle, iteration counts from 0 up, the two sides of the rule,
eager and captured and without allocation bit for bit, early stops."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _band_spd(n, reach, seed):
    """Symmetric, strictly diagonally dominant, rows i-reach .. i+reach."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), 2 * reach + 1)
    j = i + np.tile(np.arange(-reach, reach + 1), n)
    keep = (j >= 0) & (j < n)
    i, j = i[keep], j[keep]
    half = rng.uniform(-1, 1, (n, reach + 1))
    v = np.where(i == j, 2.0 * reach + 1.0, half[np.minimum(i, j), np.abs(i - j)])
    rp = np.concatenate([[0], np.cumsum(np.bincount(i, minlength=n))]).astype(np.int32)
    return gen.Csr(n, n, rp, j.astype(np.int32), v, f"band{n}w{2 * reach + 1}")


MATS = {
    "width_3": lambda: _band_spd(9001, 1, 1),
    "width_5": lambda: _band_spd(6400, 2, 2),
    "width_9": lambda: _band_spd(4097, 4, 3),
    "width_11": lambda: _band_spd(20000, 5, 4),
    "width_13": lambda: _band_spd(20000, 6, 5),          # two kernels
    "blocks_512": lambda: _band_spd(131072, 1, 6),
    "blocks_513": lambda: _band_spd(131073, 1, 7),       # two kernels
    "stencil": lambda: gen.stencil(26, 7),
}


@pytest.mark.parametrize("name", sorted(MATS))
def test_fused_cg(name):
    A = MATS[name]()
    h = L.Csr.from_gen(A, cols=A.cols)
    h.set_layout(L.LAYOUT_BAND)
    assert h.info().layout == L.LAYOUT_BAND
    b = gen.vector(A.rows, 61)
    bd = torch.from_numpy(b).to(DEV)
    for iters in (0, 1, 2, 17):
        ref, done, hist = oracle.cg(A.row_ptr, A.col_idx, A.vals, b, iters)
        xs = [torch.full((A.rows,), np.nan, dtype=torch.float64, device=DEV) for _ in range(3)]
        got = h.cg(bd, xs[0], iters, graph=False, want_result=True)
        h.cg(bd, xs[1], iters, graph=True)
        h.cg_noalloc(bd, xs[2], iters)
        torch.cuda.synchronize()
        assert torch.equal(xs[0], xs[1]) and torch.equal(xs[0], xs[2])
        scale = np.max(np.abs(ref)) if iters else 1.0
        assert np.max(np.abs(xs[0].cpu().numpy() - ref)) <= 1e-10 * scale
        assert got[1] == done == iters
        rho = float(hist[-1])
        # r.r from the recurrence: within rounding of the oracle's while it is large
        assert abs(got[0] - rho) <= 1e-8 * float(b @ b)
    # a zero right-hand side stops at once
    x = torch.full((A.rows,), np.nan, dtype=torch.float64, device=DEV)
    assert h.cg(torch.zeros_like(bd), x, 5, want_result=True) == (0.0, 0)
    assert bool((x == 0).all())
    h.destroy()


def test_two_handles_on_two_streams():
    """Solves of two handles at once, each twice: the state is the handle's."""
    A = gen.stencil(24, 7)
    hs = [L.Csr.from_gen(A, cols=A.cols) for _ in range(2)]
    b = [torch.from_numpy(gen.vector(A.rows, 70 + k)).to(DEV) for k in range(2)]
    want = [torch.empty_like(b[0]) for _ in range(2)]
    for h, bi, w in zip(hs, b, want):
        h.cg(bi, w, 30)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(2):
        got = [torch.zeros_like(b[0]) for _ in range(2)]
        torch.cuda.synchronize()
        for h, bi, g, s in zip(hs, b, got, streams):
            h.cg(bi, g, 30, stream=s)
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want))
