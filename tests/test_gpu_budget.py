"""Calls that want working memory beside what they cannot do without, where the
device budget (LILAC_HBM_BUDGET, read when the library starts: a process of its
own for each test) leaves no room for it: they run all the same."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = """
import numpy as np, torch
import gen, oracle
import paper_2001_07938_amd as L

def refused(n):
    # whether a diagonal matrix of n rows (20 bytes a row) is
    try:
        L.Csr.from_gen(gen.identity(n)).destroy()
        return False
    except L.LilacError as e:
        assert e.code == -4, e
        return True

def fill(n, step):
    # matrices of `step` rows until one of n rows no longer fits
    kept = []
    while not refused(n):
        kept.append(L.Csr.from_gen(gen.identity(step)))
    return kept
"""


def _child(budget, body):
    env = dict(os.environ, LILAC_HBM_BUDGET=str(budget))
    r = subprocess.run([sys.executable, "-c", HEAD + body + "\nprint('child ok')"], cwd=ROOT,
                       env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr


def test_pagerank_without_working_memory():
    """A matrix over renamed hot columns: x in their order (260 KB) does not fit
    beside the second vector; same result as where it does."""
    _child("160M", """
n = 65000
rng = np.random.default_rng(4)
lens = rng.integers(30, 71, n)
lens[7] = 3000
rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
A = gen.Csr(n, n, rp, rng.integers(0, n, rp[-1]).astype(np.int32),
            rng.uniform(0, 1 / 50, rp[-1]).astype(np.float32), 'wide')
def rank(h):
    x = torch.full((n,), 1.0 / n, dtype=torch.float32, device='cuda')
    return h.pagerank(0.85, 6, x).clone()
h = L.Csr.from_gen(A, cols=n)
assert h.info().layout == L.LAYOUT_HOT
want = rank(h)
h.destroy()
h = L.Csr.from_gen(A, cols=n)
kept = [fill(400000, 200000), fill(100000, 20000), fill(16000, 500)]
got = rank(h)
torch.cuda.synchronize()
assert torch.equal(got, want)
""")


def test_band_where_the_panels_do_not_fit():
    """Local columns that suit the column panels (500 lines of x to 64 rows):
    with memory for the band layout's word per entry only, that is taken."""
    _child("64M", """
A = gen.random_rows(8000, 5, 60, seed=9)
x = torch.from_numpy(gen.vector(A.cols, 1)).cuda()
h = L.Csr.from_gen(A, cols=A.cols)
assert h.info().layout == L.LAYOUT_PANELS
h.destroy()
kept = [fill(1000000, 200000), fill(165000, 3000)]
h = L.Csr.from_gen(A, cols=A.cols)
assert h.info().layout == L.LAYOUT_BAND
y = torch.empty(A.rows, dtype=torch.float64, device='cuda')
h.spmv(x, y)
from tests.helpers import TOL_F64, check_spmv
check_spmv(A, gen.vector(A.cols, 1), y.cpu().numpy(), TOL_F64)
""")


def test_pagerank_refused_again_and_again():
    """The relabelled copy of a graph does not fit: every call says so, and the
    first one with room gives the result (a copy left half made by a refused call
    would be used by the next)."""
    _child("64M", """
n = 70000
A = gen.random_rows(n, 4, 12, seed=5).astype(np.float32)
A.vals = np.abs(A.vals) / 12
def rank(h):
    x = torch.full((n,), 1.0 / n, dtype=torch.float32, device='cuda')
    return h.pagerank(0.85, 6, x).clone()
h = L.Csr.from_gen(A, cols=n)
want = rank(h)
h.destroy()
h = L.Csr.from_gen(A, cols=n)
kept = fill(800000, 200000) + fill(100000, 20000) + fill(16000, 500)
left = len(kept)
while kept:     # a little more room each time
    try:
        got = rank(h)
        break
    except L.LilacError as e:
        assert e.code == -4, e
    kept.pop().destroy()
assert 0 < len(kept) < left
torch.cuda.synchronize()
assert torch.equal(got, want)
""")


def test_solve_takes_the_same_steps_or_none():
    """The three more vectors of a solve with one kernel per iteration: where they
    do not fit the call says so; it never gives other bits than with more
    memory."""
    _child("64M", """
A = gen.stencil(32, 7)
b = torch.from_numpy(gen.vector(A.rows, 1)).cuda()
def solve(h):
    x = torch.full_like(b, float('nan'))
    h.cg(b, x, 10)
    torch.cuda.synchronize()
    return x
h = L.Csr.from_gen(A, cols=A.cols)
want = solve(h)
x = torch.full_like(b, float('nan'))
h.cg_noalloc(b, x, 10)
torch.cuda.synchronize()
assert torch.equal(x, want)
h.destroy()
h = L.Csr.from_gen(A, cols=A.cols)
# 1.5 MB left (31 bytes a row refused): four vectors (1 MB), not seven (1.8 MB)
kept = [fill(800000, 200000), fill(100000, 20000), fill(50000, 2000)]
for k in range(2):
    try:
        assert torch.equal(solve(h), want)
        assert k == 1
    except L.LilacError as e:
        assert e.code == -4 and k == 0, e
    kept.pop()
""")


def test_kept_working_memory_is_given_back():
    """What BFS (half a byte a row) and the JDS product (four) keep for their next
    call does not stand in the way of a handle that needs the room."""
    _child("96M", """
n = 4000000
A = gen.identity(n // 8)
J = L.Csr.from_gen(A, cols=A.cols)
j = J.to_jds()
x = torch.ones(A.rows, dtype=torch.float64, device='cuda')
y = torch.empty_like(x)
kept = [J] + fill(100000, 20000) + fill(16000, 500)
level = torch.empty(A.rows, dtype=torch.int32, device='cuda')
while len(kept) > 1:              # a little more room, until the call runs
    kept.pop().destroy()
    try:
        L.lilac_spmv_jds(A.rows, j['max_len'], j['perm'], j['nzcnt'], j['jd_ptr'], j['col_ind'],
                         j['val'], x, y)
        break
    except L.LilacError as e:
        assert e.code == -4, e
assert torch.equal(x, y)
# the call has kept 2 MB; some 0.6 MB are left (31 bytes a row wanted)
assert J.bfs(0, level) == 1
h = L.Csr.from_gen(gen.identity(60000))
h.destroy()
assert J.bfs(0, level) == 1
L.lilac_spmv_jds(A.rows, j['max_len'], j['perm'], j['nzcnt'], j['jd_ptr'], j['col_ind'],
                 j['val'], x, y)
assert torch.equal(x, y)
""")
