"""Set construction where its kernels can go wrong: the neighbour search with
32 lanes an atom (narrow cells with more stencil bins than lanes, several bins
an axis, a full list of 16), the counting sort over runs of several atoms per
thread (more atoms than threads, sizes that do not divide), and the float angle
tables that appear with the first float call.

Neighbours are compared with the brute-force enumeration (exact); the order by
coordination is checked through the energies and forces (float64 1e-10, float32
1e-6 eV/atom and 1e-4 eV/A, as elsewhere).
"""
import numpy as np
import pytest

import workloads as W
from oracle import tersoff as T
from oracle.neighbors import neighbor_list_set

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


def entries(i, j, sh):
    return sorted(zip(i.tolist(), j.tolist(), map(tuple, sh.tolist())))


def cases():
    # 1.9 A wide in x: 5 images a side there; a sheared cell; 1,027 atoms
    chain = np.array([[0.1, 5.0, 5.0]]), np.diag([1.9, 10.0, 10.0])
    shear = np.array([[0.2, 0.3, 0.1], [1.6, 1.4, 1.2]]), np.array([[3.5, 0, 0], [2.5, 3.4, 0], [1.0, -2.0, 3.6]])
    pos, cell = W.diamond(6, 6, 4)                                  # 1,152 sites
    keep = np.sort(rng(1).permutation(len(pos))[:1027])
    return {"narrow": [chain, shear], "vacancies": [(W.displace(rng(2), pos[keep], 0.1), cell), chain],
            "packing": [W.random_packing(rng(3), 700)]}


@pytest.mark.parametrize("name", ["narrow", "vacancies", "packing"])
def test_neighbors_and_order(api, name):
    s = W.make_set(cases()[name])
    ts = api.from_structures(s)
    assert entries(*ts.neighbors()) == entries(*neighbor_list_set(s, R2)[:3])
    x = np.asarray([W.TABLE2_X])
    ref = T.evaluate_set(s, x[0], R1, R2)
    sizes = s.sizes()
    for prec in ("fp64", "fp32", "fp64"):
        out = ts.tersoff_eval(x, precision=prec)
        E, F = out["E"][0].cpu().numpy(), out["F"][0].cpu().numpy()
        if prec == "fp64":
            assert np.abs(E - ref["E"]).max() <= 1e-10 * max(np.abs(ref["E"]).max(), 1e-2)
            assert np.abs(F - ref["F"]).max() <= 1e-10 * max(np.abs(ref["F"]).max(), 1.0)
        else:
            assert np.abs(E / sizes - ref["E"] / sizes).max() <= 1e-6
            assert np.abs(F - ref["F"]).max() <= 1e-4
    ts.close()


def test_float_tables_follow_the_geometry(api):
    """A set whose first float call comes after a float64 call and a geometry
    update, and updates after it, against sets built at the positions."""
    import ctypes

    import torch
    from paper_1909_11474_amd import _lib as L
    pos, cell = W.random_packing(rng(5), 200)
    moved = [W.displace(rng(6 + k), pos, 0.01) for k in range(2)]
    x = np.asarray([W.TABLE2_X])
    ts = api.TersoffSet(pos, cell[None], [0, len(pos)])
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    L.check(ts._lib.mt_set_list_skin(ts._handle, 0.2, st), "mt_set_list_skin")
    ts.tersoff_eval(x, precision="fp64")
    for p in moved:
        soa = torch.as_tensor(p.T.copy(), device="cuda").contiguous()
        L.check(ts._lib.mt_set_update_geometry(ts._handle, ctypes.c_void_p(soa.data_ptr()), st), "update")
        got = ts.tersoff_eval(x, precision="fp32")
        fresh = api.TersoffSet(p, cell[None], [0, len(p)])
        want = fresh.tersoff_eval(x, precision="fp64")
        assert float((got["E"] - want["E"]).abs().max()) / len(p) <= 1e-6
        assert float((got["F"] - want["F"]).abs().max()) <= 1e-4
        fresh.close()
    ts.close()
