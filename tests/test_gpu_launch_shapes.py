"""Launch shapes the other tests do not reach: every block size in whole
wavefronts (rows of one to four wavefronts in the last place of a block, which
take the costly and cheap chunks of 64 atoms in turn), and the work lists of an
open tile at small, odd and large populations, and structures of many neighbours
of which a block's LDS holds fewer replicas than its threads would; structures of
few neighbours, down to none, in the launch of a class above theirs.

Z in float64 is bit-identical to the plain schedule (one item per launch); in
float32 it is bit-identical across shapes.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


@pytest.fixture(scope="module")
def tset():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    dia, cell = W.diamond(2, 2, 2)
    s = W.make_set([W.random_packing(rng(n), n) for n in (9, 33, 100, 129, 190)] +
                   [(W.displace(rng(1), dia, 0.1), cell)])
    ts = api.from_structures(s)
    ref = ts.tersoff_eval(W.draw_params(rng(2), 1), precision="fp64")
    n = torch.as_tensor(s.sizes(), dtype=torch.float64, device="cuda")
    ts.attach_reference(ref["E"][0] / n, ref["W"][0] / n[:, None], ref["F"][0])
    yield ts
    ts.close()


@pytest.mark.parametrize("block", [192, 256, 320, 384, 448, 512])
def test_every_block_size(tset, block, tmp_path):
    X = W.draw_params(rng(3), 11)
    plain = tset.fitness(X, precision="fp64", schedule="plain").cpu().numpy()
    f32 = tset.fitness(X, precision="fp32").cpu().numpy()
    s = tset.stats()
    for prec, code, want in (("fp64", 0, plain), ("fp32", 1, f32)):
        p = tmp_path / prec
        p.write_text("N=%d S=%d nb=%d trip=%d P=%d prec=%d | block=%d tile=3 persistent=0 graph=0 ms=1\n" % (
            s["n_atoms"], s["n_struct"], s["n_bonds"], s["n_triplets"], len(X), code, block))
        tset.autotune(len(X), prec, str(p))
        got = tset.fitness(X, precision=prec).cpu().numpy()
        assert p.read_text().count("\n") == 1           # the shape was taken, not timed
        assert np.array_equal(got, want), prec


@pytest.mark.parametrize("P", [1, 2, 7, 65, 500])
def test_open_tile(tset, P):
    X = W.draw_params(rng(4), 1000)[:P]
    got = tset.fitness(X, precision="fp64").cpu().numpy()
    plain = tset.fitness(X, precision="fp64", schedule="plain").cpu().numpy()
    assert np.array_equal(got, plain)
    # each candidate's value does not depend on how many others there are
    one = tset.fitness(X[-1:], precision="fp64").cpu().numpy()
    assert np.array_equal(got[-1:], one)
    _, G = tset.fitness_grad(X, precision="fp64")
    _, g = tset.fitness_grad(X[-1:], precision="fp64")
    assert np.array_equal(G[-1:].cpu().numpy(), g.cpu().numpy())


# atoms, density (random packing, at least 1.9 A apart) and seed; 256 atoms are
# a close-packed cell, whose exchange fills more than half of a block's LDS
DENSE = [(8, 0.1, 8010), (16, 0.1, 16010), (32, 0.1, 32050), (64, 0.1, 64010), (256, None, 0)]


@pytest.mark.parametrize("n,rho,seed", DENSE)
def test_fewer_replicas_than_a_block_has_threads_for(n, rho, seed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    if rho is None:
        grid = np.array([[i, j, k] for i in range(4) for j in range(4) for k in range(4)], dtype=float)
        base = 0.5 * np.array([[0, 0, 0], [0, 1, 1], [1, 0, 1], [1, 1, 0]])
        a = 2.95 * np.sqrt(2.0)
        dense = (W.displace(rng(1), (grid[:, None] + base[None]).reshape(-1, 3) * a, 0.02), np.eye(3) * 4 * a)
    else:
        dense = W.random_packing(rng(seed), n, rho=rho, dmin=1.9)
    s = W.make_set([W.random_packing(rng(9), 9), dense])
    X = W.draw_params(rng(3), 70)
    ts = api.from_structures(s)
    kmax = ts.stats()["max_coordination"]
    assert 512 * kmax * 32 > 160 * 1024              # bytes of exchange of a full block
    ref = ts.tersoff_eval(X[:1], precision="fp64")
    m = torch.as_tensor(s.sizes(), dtype=torch.float64, device="cuda")
    ts.attach_reference(ref["E"][0] / m, ref["W"][0] / m[:, None], ref["F"][0])
    for P in (1, 7, 70):
        got = ts.fitness(X[:P], precision="fp64").cpu().numpy()
        plain = ts.fitness(X[:P], precision="fp64", schedule="plain").cpu().numpy()
        assert np.array_equal(got, plain), P
    ts.close()


@pytest.mark.parametrize("P", [1, 3, 40])
def test_few_neighbours_in_the_launch_of_a_larger_class(P):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    box, c = 20.0 * np.eye(3), np.array([10.0, 10.0, 10.0])
    tri = np.array([[0, 0, 0], [1, 0, 0], [0.5, np.sqrt(3) / 2, 0]])
    line = np.array([[2.4 * k, 0.0, 0.0] for k in range(70)])      # more than one wavefront of dimers and a chain
    s = W.make_set([(c[None], box), (c + 2.4 * tri[:2], box), (c + 2.4 * tri, box),
                    (line + 10.0, np.diag([200.0, 20.0, 20.0])), W.diamond(1, 1, 1), W.diamond(2, 2, 2),
                    W.random_packing(rng(64), 64)])
    X = W.draw_params(rng(5), P)
    ts = api.from_structures(s)
    assert ts.stats()["max_coordination"] > 4
    ref = ts.tersoff_eval(W.draw_params(rng(6), 1), precision="fp64")
    m = torch.as_tensor(s.sizes(), dtype=torch.float64, device="cuda")
    ts.attach_reference(ref["E"][0] / m, ref["W"][0] / m[:, None], ref["F"][0])
    plain = ts.tersoff_eval(X, precision="fp64", schedule="plain")
    got = ts.tersoff_eval(X, precision="fp64")
    for k in plain:
        assert torch.equal(got[k], plain[k]), k
    assert torch.equal(ts.fitness(X, precision="fp64"), ts.fitness(X, precision="fp64", schedule="plain"))
    _, G = ts.fitness_grad(X, precision="fp64")
    one = torch.cat([ts.fitness_grad(X[k:k + 1], precision="fp64")[1] for k in range(P)])
    many = ts.fitness_grad(np.repeat(X, 400, 0), precision="fp64")[1][::400]    # class 4 in a launch of its own
    assert torch.equal(G, one) and torch.equal(G, many)
    ts.close()
