"""Position updates inside captured graphs and the float path's angle tables, which
follow the geometry: a float call after a replay gives the bits of a set whose
geometry was updated outside of a graph.  One set below and one above six
neighbours (only the latter has angular moments).
"""
import ctypes

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

OUT = ("E", "F", "W")


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def make_pair(pos, cell, above_six):
    """Two sets of one displaced structure, their positions and two later ones."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api, _lib as L
    s = W.make_set([(pos, cell)])
    p = [torch.as_tensor(np.ascontiguousarray(q.T), device="cuda")
         for q in (s.pos, W.displace(rng(3), s.pos, 0.02), W.displace(rng(4), s.pos, 0.02))]
    sets = []
    for _ in range(2):
        ts = api.from_structures(s)
        L.check(ts._lib.mt_set_list_skin(ts._handle, ctypes.c_double(0.2), None), "skin")
        sets.append(ts)
    assert (sets[0].stats()["max_coordination"] > 6) == above_six
    torch.cuda.synchronize()
    return (*sets, p)


def update(ts, pos, stream=None):
    import torch
    from paper_1909_11474_amd import _lib as L
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    L.check(ts._lib.mt_set_update_geometry(ts._handle, ptr(pos), st), "geometry")


def same(a, b):
    import torch
    torch.cuda.synchronize()
    return all(torch.equal(a[k], b[k]) for k in OUT)


@pytest.mark.parametrize("above_six", [False, True])
def test_captured_update_before_any_float_call(above_six):
    import torch
    pos, cell = W.random_packing(rng(1), 100) if above_six else W.diamond(2, 2, 2)
    ts, eager, (p0, p1, p2) = make_pair(pos, cell, above_six)
    X = W.draw_params(rng(5), 3)
    buf = p0.clone()
    double = ts.eval_call(X, precision="fp64")
    double()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        update(ts, buf)
        double()
    want = {}
    for k, p in enumerate((p0, p1, p2)):
        update(eager, p)
        want[k] = {n: t.clone() for n, t in eager.tersoff_eval(X, precision="fp32").items() if n in OUT}
    assert same(ts.tersoff_eval(X, precision="fp32"), want[0])   # the tables are built here
    for k, p in ((1, p1), (2, p2), (1, p1)):
        buf.copy_(p)
        g.replay()
        assert same(ts.tersoff_eval(X, precision="fp32"), want[k]), k
    del g
    ts.close()
    eager.close()


@pytest.mark.parametrize("above_six", [False, True])
def test_first_float_call_in_the_graph(above_six):
    """640 atoms: the two-pass path, whose first float call allocates nothing after a
    float64 one and so can be captured."""
    import torch
    pos, cell = W.diamond(4, 4, 5)
    pos = W.displace(rng(1), pos, 0.25 if above_six else 0.05)
    ts, eager, (p0, p1, p2) = make_pair(pos, cell, above_six)
    X = W.draw_params(rng(6), 3)
    want = {}
    for k, p in enumerate((p0, p1, p2)):
        update(eager, p)
        want[k] = {n: t.clone() for n, t in eager.tersoff_eval(X, precision="fp32").items() if n in OUT}
    call = ts.eval_call(X, precision="fp32")
    buf = p0.clone()
    ts.tersoff_eval(X, precision="fp64")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        update(ts, buf)
        call()
        update(ts, buf)
        call()
    assert same(ts.tersoff_eval(X, precision="fp32"), want[0])   # before any replay
    for k, p in ((1, p1), (2, p2), (0, p0)):
        buf.copy_(p)
        g.replay()
        torch.cuda.synchronize()
        got = {"E": call.E, "F": call.F.transpose(1, 2), "W": call.W}
        assert same(got, want[k]), k
        assert same(ts.tersoff_eval(X, precision="fp32"), want[k]), k
    del g
    ts.close()
    eager.close()
