"""fitness_eval by captured graph (a launch shape with graph=1): replays give the bits
of the direct launches of the same shape, follow new parameters in the bound buffer, and are
captured again where a buffer that they hold has moved.
"""
import numpy as np
import pytest

import workloads as W
from oracle import tersoff as T

pytestmark = pytest.mark.gpu

R1, R2 = 2.8, 3.2


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api as A
    return A


def use_shape(ts, P, precision, path, graph, block=512, tile=8):
    st = ts.stats()
    path.write_text("N=%d S=%d nb=%d trip=%d P=%d prec=%d | block=%d tile=%d persistent=0 graph=%d ms=0\n" % (
        st["n_atoms"], st["n_struct"], st["n_bonds"], st["n_triplets"], P, precision == "fp32", block, tile, graph))
    ts.autotune(P, precision, str(path))
    assert path.read_text().count("\n") == 1            # the shape was taken, not timed


def with_refs(api, s, seed):
    refs = T.reference_data(s, W.draw_params(rng(seed), 1)[0], R1, R2)
    ts = api.from_structures(s)
    ts.attach_reference(refs["e"], refs["w"], refs["f"])
    return ts


def close_packed(n, a):
    base = np.array([[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]])
    grid = np.array([[i, j, k] for i in range(n) for j in range(n) for k in range(n)], dtype=float)
    return (grid[:, None] + base[None]).reshape(-1, 3) * a, np.eye(3) * n * a


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx", [6, 9])
@pytest.mark.parametrize("kind", ["batched", "large", "lds"])
def test_replays_and_moving_buffers(api, tmp_path, kind, nx, precision):
    """batched: cells and packings; large: beside a 600-atom packing (staging buffer);
    lds: beside a 500-atom close-packed cell, which in float64 exceeds a block's LDS
    (block sums of its two-pass launches in a buffer of their own)."""
    import torch
    first = {"batched": lambda: W.random_packing(rng(1), 100), "large": lambda: W.random_packing(rng(1), 600),
             "lds": lambda: close_packed(5, 2.95 * np.sqrt(2.0))}[kind]()
    s = W.make_set([(W.displace(rng(2), first[0], 0.02), first[1])] + W.strained_diamond_cells(3, 3))
    ts = with_refs(api, s, 4)
    draw = W.draw_params if nx == 6 else W.draw_params_full
    P = 6
    pops = [draw(rng(5 + k), P) for k in range(3)]
    use_shape(ts, P, precision, tmp_path / "direct", 0)
    want = [ts.fitness(x, precision=precision).clone() for x in pops]
    use_shape(ts, P, precision, tmp_path / "graph", 1)
    X = torch.as_tensor(pops[0], device="cuda").contiguous()
    Z = torch.empty(P, 4, dtype=torch.float64, device="cuda")
    call = ts.fitness_call(X, Z, precision=precision)

    def check():
        for k in (0, 1, 2, 0):
            X.copy_(torch.as_tensor(pops[k]))
            Z.fill_(-1.0)
            call()
            torch.cuda.synchronize()
            assert torch.equal(Z, want[k]), k

    check()
    ts.fitness(draw(rng(9), 60), precision="fp64")      # larger buffers, freed ones under the graph
    check()
    ts.tersoff_eval(draw(rng(10), 70), precision="fp64")
    check()
    other = 15 - nx
    xo = (W.draw_params if other == 6 else W.draw_params_full)(rng(11), P)
    a = ts.fitness(xo, precision=precision).clone()     # the other form's graph
    check()
    assert torch.equal(ts.fitness(xo, precision=precision), a)
    ts.close()


def test_more_buffers_than_graphs_are_kept(api, tmp_path):
    """Sixteen graphs are kept; the twentieth pair of buffers takes the oldest's place."""
    import torch
    s = W.make_set(W.strained_diamond_cells(3, 4))
    ts = with_refs(api, s, 4)
    P = 3
    pops = [torch.as_tensor(W.draw_params(rng(20 + k), P), device="cuda") for k in range(20)]
    want = [ts.fitness(x).clone() for x in pops]
    use_shape(ts, P, "fp32", tmp_path / "graph", 1)
    calls = [ts.fitness_call(x, torch.empty(P, 4, dtype=torch.float64, device="cuda")) for x in pops]
    for _ in range(2):
        for c, z in zip(calls, want):
            c()
            torch.cuda.synchronize()
            assert torch.equal(c.Z, z)
    ts.close()


def test_graph_after_a_position_update(api, tmp_path):
    """A float graph made before the float tables followed new positions: an update
    that keeps the layout, then new references (which drop the graphs)."""
    import ctypes
    import torch
    from paper_1909_11474_amd import _lib as L
    s = W.make_set(W.strained_diamond_cells(3, 3))
    moved = W.displace(rng(30), s.pos, 0.01)
    s1 = W.make_set([(moved[s.offset[k]:s.offset[k + 1]], s.cell[k]) for k in range(s.n_struct)])
    refs = T.reference_data(s1, W.draw_params(rng(4), 1)[0], R1, R2)
    fresh = api.from_structures(s1)
    fresh.attach_reference(refs["e"], refs["w"], refs["f"])
    ts = with_refs(api, s, 4)
    X = torch.as_tensor(W.draw_params(rng(31), 5), device="cuda")
    want = fresh.fitness(X)
    use_shape(ts, 5, "fp32", tmp_path / "graph", 1)
    Z = torch.empty(5, 4, dtype=torch.float64, device="cuda")
    call = ts.fitness_call(X, Z)
    call()
    pos = torch.as_tensor(np.ascontiguousarray(moved.T), device="cuda")
    torch.cuda.synchronize()
    L.check(ts._lib.mt_set_update_positions(ts._handle, ctypes.c_void_p(pos.data_ptr()), None), "update")
    ts.attach_reference(refs["e"], refs["w"], refs["f"])
    for _ in range(3):
        Z.fill_(-1.0)
        call()
        torch.cuda.synchronize()
        assert torch.equal(Z, want)
    fresh.close()
    ts.close()
