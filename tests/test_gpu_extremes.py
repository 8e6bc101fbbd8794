"""Parameters at the ends of the domain: intermediate values of a candidate that
leave the range of the arithmetic type, or a zeta near its smallest value.

The expected values are those of the limit that the formulas have there:
  d -> large:  g^T -> gamma, so a candidate of d = 1e200 (1e30 in float32, where
               d^2 already overflows) equals one whose d is large but whose d^2 is
               still in range, up to terms of c^2 / d^2 < 1e-30: same tolerance as
               for equal candidates (1e-12 of the largest value in float64, where
               the gradient's sums round differently; 1e-6 in float32).
  zeta^n -> inf: b = 0.
  beta small:  zeta^n is of order 0.02 at n = 0.05, beta = 1e-33, and the forces
               depend on it; float32 against the oracle within 1e-4 eV/A.
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


@pytest.fixture(scope="module")
def structs():
    """A cell of 4 neighbours, a packing above 6, and a block on the two-pass path."""
    pos, cell = W.diamond(2, 2, 2)
    big, bcell = W.diamond(4, 4, 5)
    return W.make_set([(W.displace(rng(1), pos, 0.1), cell), W.random_packing(rng(2), 60),
                       (W.displace(rng(3), big, 0.1), bcell)])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_large_d(api, structs, precision):
    ts = api.from_structures(structs)
    far, near = (1e200, 1e120) if precision == "fp64" else (1e30, 1e16)
    X = np.repeat(W.draw_params_full(rng(4), 1), 2, axis=0)
    X[:, 6] = 1.0
    X[:, 7] = far, near
    out = {k: v.cpu().numpy() for k, v in ts.tersoff_eval(X, precision=precision).items()}
    tol = 1e-12 if precision == "fp64" else 1e-6
    for k in ("E", "F", "W"):
        assert np.isfinite(out[k]).all(), k
        assert np.abs(out[k][0] - out[k][1]).max() <= tol * np.abs(out[k][1]).max(), k
    refs = T.reference_data(structs, W.draw_params_full(rng(5), 1)[0], R1, R2)
    ts.attach_reference(refs["e"], refs["w"], refs["f"])
    Z, G = (t.cpu().numpy() for t in ts.fitness_grad(X, precision=precision))
    assert np.isfinite(Z).all() and np.isfinite(G).all(), G
    assert np.abs(Z[0] - Z[1]).max() <= tol * np.abs(Z[1]).max()
    assert np.abs(G[0] - G[1]).max() <= tol * np.abs(G[1]).max()
    ts.close()


def test_zeta_power_overflow(api, structs):
    """zeta^n beyond the largest double: b = (1 + inf)^(-1/(2n)) = 0, so the energy
    is the repulsive part alone (float64; the forces have no finite value)."""
    ts = api.from_structures(structs)
    x = np.array(W.TABLE2_X)
    x[3], x[4] = 1e200, 50.0
    E = ts.tersoff_eval(x[None], precision="fp64")["E"].cpu().numpy()[0]
    # U = 1/2 sum f_C (f_R - b f_A), b = 1 for an atom's only bond
    want = np.zeros(len(structs.sizes()))
    from oracle.neighbors import neighbor_list
    for k in range(structs.n_struct):
        pos, cell = structs.structure(k)
        i, j, sh = neighbor_list(pos, cell, R2)
        r = np.linalg.norm(pos[j] + sh @ cell - pos[i], axis=1)
        fc = np.where(r <= R1, 1.0, 0.5 * (1.0 + np.cos(np.pi * (r - R1) / (R2 - R1))))
        b = np.bincount(i, minlength=len(pos))[i] == 1
        e = np.exp(-x[1] * (r - x[2]))
        want[k] = 0.5 * (fc * x[0] * (e * e - 2.0 * b * e)).sum()
    assert np.abs(E - want).max() <= 1e-10 * np.abs(want).max(), (E, want)
    ts.close()


def test_small_zeta_float(api, structs):
    ts = api.from_structures(structs)
    x = np.array(W.TABLE2_X)
    x[3], x[4] = 1e-33, 0.05
    out = ts.tersoff_eval(x[None], precision="fp32")
    ref = T.evaluate_set(structs, x, R1, R2)
    F = out["F"].cpu().numpy()[0]
    assert np.abs(F - ref["F"]).max() <= 1e-4, np.abs(F - ref["F"]).max()
    n = structs.sizes().astype(float)
    assert np.abs(out["E"].cpu().numpy()[0] / n - ref["E"] / n).max() <= 1e-6
    ts.close()
