"""The vector update of a CG iteration by pairs (more than 262,144 rows): sizes
around the bound and around whole pairs and rounds, a last odd element, a
solution that starts off a 16-byte bound, early stops."""
import numpy as np
import pytest
import torch

import gen
import oracle
import paper_2001_07938_amd as L
from tests.test_gpu_cg_fused import _band_spd

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", (262143, 262144, 262145, 262147, 524289, 1048576, 1048579))
def test_step_sizes(n):
    A = _band_spd(n, 1, n)
    h = L.Csr.from_gen(A, cols=n)
    b = gen.vector(n, 62)
    bd = torch.from_numpy(b).to(DEV)
    for iters in (1, 6):
        ref, done, hist = oracle.cg(A.row_ptr, A.col_idx, A.vals, b, iters)
        x = torch.full((n + 1,), np.nan, dtype=torch.float64, device=DEV)
        got = h.cg(bd, x[:n], iters, graph=False, want_result=True)
        # iteration by iteration the dot products differ by rounding only
        assert np.max(np.abs(x[:n].cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref))
        assert got[1] == done == iters
        assert abs(got[0] - float(hist[-1])) <= 1e-8 * float(b @ b)
        off = torch.full((n + 1,), np.nan, dtype=torch.float64, device=DEV)
        h.cg(bd, off[1:], iters, graph=False)
        assert torch.equal(off[1:], x[:n])
        h.cg(bd, off[1:], iters, graph=True)
        assert torch.equal(off[1:], x[:n])
        assert bool(torch.isnan(x[n])) and bool(torch.isnan(off[0]))
        if n <= 1 << 20:
            h.cg_noalloc(bd, off[1:], iters)
            torch.cuda.synchronize()
            assert torch.equal(off[1:], x[:n])
    assert h.cg(torch.zeros_like(bd), x[:n], 3, want_result=True) == (0.0, 0)
    assert bool((x[:n] == 0).all())
    h.destroy()
