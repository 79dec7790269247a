"""Sums of the sliced form against exact ones: a row is added up in parts, so its
error is bounded by the roundings on the way of one entry, not by its length.  The
values make a sum in order lose every entry but the first (each is less than half
a unit in the last place of the running sum)."""
import math

import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _roundings(width):
    # two products to a sum, four sums to eight entries, four such parts, the parts
    # of 32 before, the entries past the last eight
    return 2 + 2 + 4 + (width + 31) // 32 + 2


@pytest.mark.parametrize("width", [8, 11, 16, 27, 31, 33, 64, 100, 200])
def test_sums_in_parts(width):
    rows = 65536 + 64
    rng = np.random.default_rng(width)
    i = np.repeat(np.arange(rows), width)
    j = np.clip(i + np.tile(np.arange(width), rows) - width // 2, 0, rows - 1)
    v = rng.uniform(0.5, 0.95, rows * width) * U
    v[::width] = 1.0
    A = gen.Csr(rows, rows, (np.arange(rows + 1) * width).astype(np.int32), j.astype(np.int32), v,
                f"parts{width}")
    h = L.Csr.from_gen(A, cols=rows)
    inf = h.info()
    assert inf.layout == L.LAYOUT_BAND
    assert inf.device_bytes > A.nnz * 22      # slices: a copy of the values
    y = torch.empty(rows, dtype=torch.float64, device="cuda")
    h.spmv(torch.ones(rows, dtype=torch.float64, device="cuda"), y)
    got = y.cpu().numpy()
    for r in range(0, rows, 97):
        row = v[r * width:(r + 1) * width]
        err = abs(math.fsum(np.append(row, -got[r])))
        assert err <= _roundings(width) * U * math.fsum(row) * (1 + 1e-12), (r, err / U)
    h.destroy()
