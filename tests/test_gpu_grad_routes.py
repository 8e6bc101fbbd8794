"""The fitness gradient where its work list differs from the fitness call's.

A 500-atom close-packed cell (12 neighbours per atom) needs 196 KB of exchange
slots per replica in float64, more than a block's LDS, so the float64 fitness
evaluates it by the two-pass path and writes no residuals for it; the adjoint,
which only needs 16 KB for it, has to follow (two-pass adjoint).  In float32
(98 KB) both batch it.  Beside it: a 64-atom cell (pair sums), trimers and a
dimer (zeta = 0: every derivative of b is dropped).

Tolerances as in the other gradient tests: 1e-10 (float64) and 1e-4 (float32)
of the largest component.
"""
import numpy as np
import pytest

import workloads as W
from oracle import tersoff as T

pytestmark = pytest.mark.gpu

R1, R2 = 2.8, 3.2


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def close_packed(n, a):
    base = np.array([[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]])
    grid = np.array([[i, j, k] for i in range(n) for j in range(n) for k in range(n)], dtype=float)
    return (grid[:, None] + base[None]).reshape(-1, 3) * a, np.eye(3) * n * a


@pytest.mark.parametrize("nx", [6, 9])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_gradient_follows_the_fitness_route(precision, nx):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    pos, cell = close_packed(5, 2.95 * np.sqrt(2.0))
    dia, dcell = W.diamond(2, 2, 2)
    box, c = np.eye(3) * 20.0, np.array([10.0, 10.0, 10.0])
    tri = c + 2.4 * np.array([[0, 0, 0], [1, 0, 0], [0.5, np.sqrt(3) / 2, 0]])
    s = W.make_set([(W.displace(rng(1), pos, 0.02), cell), (W.displace(rng(2), dia, 0.1), dcell),
                    (tri, box), (c + np.array([[0, 0, 0], [2.9, 0, 0]]), box)])
    draw = W.draw_params if nx == 6 else W.draw_params_full
    X, hidden = draw(rng(3), 2), draw(rng(4), 1)[0]
    refs = T.reference_data(s, hidden, R1, R2)
    ts = api.from_structures(s)
    assert ts.stats()["max_coordination"] == 12 and ts.stats()["n_large"] == 0
    ts.attach_reference(refs["e"], refs["w"], refs["f"])
    Zo, Go = T.fitness_grad(s, X, refs, (1.0, 0.7, 1.3))
    Z, G = (t.cpu().numpy() for t in ts.fitness_grad(X, (1.0, 0.7, 1.3), precision=precision))
    tol = 1e-10 if precision == "fp64" else 1e-4
    for k in range(len(X)):
        assert np.abs(G[k] - Go[k]).max() <= tol * np.abs(Go[k]).max(), (k, G[k], Go[k])
    assert np.allclose(Z, Zo, rtol=1e-10 if precision == "fp64" else 1e-5)
    ts.close()
