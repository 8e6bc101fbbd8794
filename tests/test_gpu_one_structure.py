"""Evaluation of a set of one large structure (blocks of one or four wavefronts
by its size, sums finished by the gather kernel) against the same structure
beside another one (blocks of four, sums by the finalize kernel).

Per-atom results do not depend on the blocks: the same bits.  The totals are sums
of N per-atom terms in another order: within N 2^-53 of N times the largest term
(8 N 2^-53 with the rounding of the blocks' own trees).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


# 16,384 and 65,536 are the largest sizes of one rule each; 640 leaves a
# wavefront's remainder, 74,088 a block's
@pytest.mark.parametrize("dims,P", [((4, 4, 5), 1), ((4, 4, 5), 3), ((8, 16, 16), 1), ((9, 16, 16), 1),
                                    ((16, 16, 32), 1), ((21, 21, 21), 1), ((9, 16, 16), 5)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_same_results_alone_and_beside_another(dims, P, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    pos, cell = W.diamond(*dims)
    big = (W.displace(rng(1), pos, 0.1), cell)
    small = W.diamond(2, 2, 2)
    N = len(pos)
    X = W.draw_params(rng(2), P)
    vel = np.zeros((N + len(small[0]), 3))
    vel[:N] = rng(3).normal(0.0, 0.01, size=(N, 3))
    one = api.from_structures(W.make_set([big]))
    two = api.from_structures(W.make_set([big, small]))
    assert one.stats()["n_large"] == 1 and two.stats()["n_large"] == 1
    kw = dict(precision=precision, atom_virial=True)
    a = {k: v.cpu().numpy() for k, v in one.tersoff_eval(X, velocities=vel[:N], **kw).items()}
    b = {k: v.cpu().numpy() for k, v in two.tersoff_eval(X, velocities=vel, **kw).items()}
    assert np.array_equal(a["F"], b["F"][:, :N]) and np.array_equal(a["Wi"], b["Wi"][:, :N])
    eps, wi = 8.0 * N * 2.0 ** -53, np.abs(a["Wi"]).max()
    assert np.abs(a["E"][:, 0] - b["E"][:, 0]).max() <= eps * np.abs(a["E"]).max()
    assert np.abs(a["W"][:, 0] - b["W"][:, 0]).max() <= eps * N * wi
    assert np.abs(a["J"] - b["J"]).max() <= eps * N * 3 * wi * np.abs(vel).max()
    one.close()
    two.close()
