"""Dense dot product at the edges of its split: one workgroup against many
(16384 elements), whole and cut 16-byte pieces, vectors that start off a
16-byte bound."""
import math

import numpy as np
import pytest
import torch

import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu

SIZES = (1, 2, 3, 5, 1023, 4097, 8193, 16383, 16384, 16385, 16387, 262145, 2_097_155)


@pytest.mark.parametrize("dtype", (np.float64, np.float32))
@pytest.mark.parametrize("n", SIZES)
def test_dot_edges(n, dtype):
    rng = np.random.default_rng(n)
    a = rng.standard_normal(n).astype(dtype)
    b = rng.standard_normal(n).astype(dtype)
    prod = a.astype(np.longdouble) * b.astype(np.longdouble)
    ref, mag = math.fsum(prod.astype(np.float64)), float(np.abs(prod).sum())
    # n products and sums in binary64, then one rounding of a float32 result
    eps = np.finfo(np.float64).eps
    tol = (n + 2) * eps * mag + (np.finfo(np.float32).eps * abs(ref) if dtype == np.float32 else 0)
    out = torch.empty(1, dtype=torch.float64 if dtype == np.float64 else torch.float32,
                      device="cuda")
    first = None
    for shift_a, shift_b in ((0, 0), (1, 0), (0, 1), (1, 1), (2, 3)):
        da = torch.zeros(n + 4, dtype=out.dtype, device="cuda")
        db = torch.zeros(n + 4, dtype=out.dtype, device="cuda")
        da[shift_a:shift_a + n] = torch.from_numpy(a).cuda()
        db[shift_b:shift_b + n] = torch.from_numpy(b).cuda()
        L.lilac_dot_dev(n, da[shift_a:shift_a + n], db[shift_b:shift_b + n], out)
        got = float(out.item())
        assert abs(got - ref) <= tol
        first = got if first is None else first
        assert got == first     # the start of a vector does not change the sum


def test_dot_not_finite():
    """Elements past the end and other pieces do not leak into the sum."""
    for n in (7, 16390):
        a = torch.ones(n + 9, dtype=torch.float64, device="cuda")
        a[n:] = float("nan")
        out = torch.empty(1, dtype=torch.float64, device="cuda")
        L.lilac_dot_dev(n, a, a, out)
        assert float(out.item()) == n
        a[n - 1] = float("inf")
        L.lilac_dot_dev(n, a, a, out)
        assert math.isinf(float(out.item()))
        a[0] = float("nan")
        L.lilac_dot_dev(n, a, a, out)
        assert math.isnan(float(out.item()))
