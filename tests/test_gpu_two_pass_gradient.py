"""The two-pass fitness gradient (a structure over 512 atoms) at the coordinations
where its kernels change: up to 4, 5-6 (pair sums), 7-8 and above (float: sums from
the set's table of angular moments, which only sets above six neighbours have).

Tolerances as in the other gradient tests: 1e-10 (float64) and 1e-4 (float32) of
the largest component.
"""
import ctypes

import numpy as np
import pytest

import workloads as W
from oracle import tersoff as T

pytestmark = pytest.mark.gpu

R1, R2 = 2.8, 3.2
# a displaced 640-atom diamond block's largest coordination by (displacement, seed)
BLOCK = {4: (0.08, 1), 5: (0.15, 1), 6: (0.2, 1), 7: (0.25, 1), 8: (0.25, 2), 10: (0.35, 1)}


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def block(kmax):
    sigma, seed = BLOCK[kmax]
    pos, cell = W.diamond(4, 4, 5)
    return W.make_set([(W.displace(rng(seed), pos, sigma), cell)])


def check(ts, s, kmax, nx, precision):
    st = ts.stats()
    assert st["n_large"] == 1 and st["max_coordination"] == kmax
    draw = W.draw_params if nx == 6 else W.draw_params_full
    refs = T.reference_data(s, draw(rng(60), 1)[0], R1, R2)
    ts.attach_reference(refs["e"], refs["w"], refs["f"])
    X, w = draw(rng(61), 2), (1.0, 0.7, 1.3)
    Z, G = (t.cpu().numpy() for t in ts.fitness_grad(X, w, precision=precision))
    Zo, Go = T.fitness_grad(s, X, refs, w, topology=T.topology(s, R2))
    tol = 1e-10 if precision == "fp64" else 1e-4
    for c in range(len(X)):
        assert np.abs(G[c] - Go[c]).max() <= tol * np.abs(Go[c]).max(), (c, G[c], Go[c])
    assert np.abs(Z - Zo).max() <= (1e-10 if precision == "fp64" else 1e-5) * np.abs(Zo).max()


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api as A
    return A


@pytest.mark.parametrize("kmax", sorted(BLOCK))
@pytest.mark.parametrize("nx", [6, 9])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_every_coordination_step(api, precision, nx, kmax):
    s = block(kmax)
    ts = api.from_structures(s)
    check(ts, s, kmax, nx, precision)
    ts.close()


@pytest.mark.parametrize("first,then", [(8, 5), (10, 6), (6, 8)])
def test_coordination_changes_in_a_position_update(api, first, then):
    """The moment table of the former positions must not serve the new ones."""
    import torch
    from paper_1909_11474_amd import _lib as L
    s0, s = block(first), block(then)
    ts = api.from_structures(s0)
    check(ts, s0, first, 6, "fp32")
    pos = torch.as_tensor(np.ascontiguousarray(s.pos.T), device="cuda")
    torch.cuda.synchronize()
    L.check(ts._lib.mt_set_update_positions(ts._handle, ctypes.c_void_p(pos.data_ptr()), None), "update")
    check(ts, s, then, 6, "fp32")
    ts.close()
