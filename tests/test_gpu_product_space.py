"""Products that use working memory of the handle (groups of panels, renamed hot
columns): one handle on many streams at once, streams that are gone, no
allocation in a product, an eager product while another stream is captured."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import gen
import paper_2001_07938_amd as L

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _hubs(rows, cols, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 30, rows)
    lens[77] = 3000
    rp = np.concatenate([[0], np.cumsum(lens)])
    c = rng.permutation(cols)[(cols * rng.random(rp[-1]) ** 4).astype(np.int64)]
    return gen.Csr(rows, cols, rp.astype(np.int32), c.astype(np.int32),
                   rng.uniform(-1, 1, rp[-1]), "hubs")


MATS = {"groups": (lambda: gen.random_rows(100000, 5, 60, seed=1), L.LAYOUT_PANELS),
        "hot": (lambda: _hubs(260000, 300000, 2), L.LAYOUT_HOT)}


@pytest.fixture(params=sorted(MATS))
def case(request):
    A = MATS[request.param][0]()
    h = L.Csr.from_gen(A, cols=A.cols)
    assert h.info().layout == MATS[request.param][1]
    xs = [torch.from_numpy(gen.vector(A.cols, 50 + k)).to(DEV) for k in range(12)]
    want = []
    for x in xs:
        y = torch.empty(A.rows, dtype=torch.float64, device=DEV)
        h.spmv(x, y)
        torch.cuda.synchronize()
        want.append(y)
    yield h, xs, want
    h.destroy()


def test_one_handle_on_many_streams(case):
    h, xs, want = case
    streams = [torch.cuda.Stream() for _ in xs]
    for _ in range(3):
        got = [torch.full_like(want[0], float("nan")) for _ in xs]
        torch.cuda.synchronize()
        for _ in range(4):
            for x, y, s in zip(xs, got, streams):
                h.spmv(x, y, stream=s)
        torch.cuda.synchronize()
        for y, w in zip(got, want):
            assert torch.equal(y, w)


def test_from_several_threads(case):
    h, xs, want = case
    got = [torch.full_like(want[0], float("nan")) for _ in xs]
    torch.cuda.synchronize()

    def work(k):
        s = torch.cuda.Stream()
        for _ in range(10):
            h.spmv(xs[k], got[k], stream=s)
        s.synchronize()
    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for y, w in zip(got[:4], want):
        assert torch.equal(y, w)


def test_streams_that_are_gone(case):
    """Each product on a new stream, destroyed before the next one is asked for
    (it may come at the same address)."""
    h, xs, want = case
    hip = ctypes.CDLL("libamdhip64.so")
    got = [torch.full_like(want[0], float("nan")) for _ in xs]
    torch.cuda.synchronize()
    for k, x in enumerate(xs):
        s = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0   # non-blocking
        h.spmv(x, got[k], stream=s.value)
        assert hip.hipStreamDestroy(s) == 0
    torch.cuda.synchronize()
    for y, w in zip(got, want):
        assert torch.equal(y, w)


def test_no_allocation_in_a_product(case):
    h, xs, want = case
    y = torch.empty_like(want[0])
    streams = [torch.cuda.Stream() for _ in range(10)]
    torch.cuda.synchronize()
    for s in streams:
        h.spmv(xs[0], want[0], stream=s)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for s in streams:
        for x in xs:
            h.spmv(x, y, stream=s)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free


def test_eager_product_while_another_stream_is_captured(case):
    """The first product of a handle on a stream, during a capture in the global
    mode on another: the capture goes on, both results are right."""
    h, xs, want = case
    s = torch.cuda.Stream()
    g, a, b = torch.cuda.CUDAGraph(), torch.ones(1000, device=DEV), torch.zeros(1000, device=DEV)
    y = torch.full_like(want[0], float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.graph(g):     # global mode
        b.add_(a)
        h.spmv(xs[1], y, stream=s)
        b.add_(a)
    torch.cuda.synchronize()
    assert torch.equal(y, want[1])
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(b, torch.full_like(b, 2.0 * (k + 1)))
