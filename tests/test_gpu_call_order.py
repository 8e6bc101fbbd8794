"""The same bits whatever kernels ran before: lanes outside a structure and registers
that were spilled hold nothing from earlier launches.  Structures of 17, 16, 54 and 30
atoms (lanes of a group and of a wavefront without an atom) of up to 16 neighbours.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_edges import bcc_cell, shell16

pytestmark = pytest.mark.gpu


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def test_every_order_gives_the_same_bits():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    s = W.make_set([shell16(), bcc_cell(rng(1), 2), bcc_cell(rng(2), 3), W.random_packing(rng(3), 30),
                    W.diamond(1, 1, 1)])
    ts = api.from_structures(s)
    assert ts.stats()["max_coordination"] == 16
    ref = ts.tersoff_eval(W.draw_params(rng(4), 1), precision="fp64")
    n = torch.as_tensor(s.sizes(), dtype=torch.float64, device="cuda")
    ts.attach_reference(ref["E"][0] / n, ref["W"][0] / n[:, None], ref["F"][0])
    vel = rng(5).normal(0.0, 0.01, size=(len(s.pos), 3))
    calls = []
    for nx, draw in ((6, W.draw_params), (9, W.draw_params_full)):
        for p in ("fp64", "fp32"):
            x = draw(rng(6), 3)
            calls += [lambda x=x, p=p: list(ts.tersoff_eval(x, precision=p, atom_virial=True).values()),
                      lambda x=x, p=p: list(ts.tersoff_eval(x, precision=p, velocities=vel).values()),
                      lambda x=x, p=p: [ts.fitness(x, precision=p)],
                      lambda x=x, p=p: [ts.fitness(x, precision=p, schedule="plain")],
                      lambda x=x, p=p: list(ts.fitness_grad(x, precision=p))]
    first = [[t.clone() for t in c()] for c in calls]
    assert all(torch.isfinite(t).all() for f in first for t in f)
    for turn in range(3):
        for k in rng(turn).permutation(len(calls)):
            for a, b in zip(calls[k](), first[k]):
                assert torch.equal(a, b), k
    ts.close()
