"""The first half of a step in one kernel against kick, drift and displacement
check one after another (the same bits), and the kinetic sums against float64
sums on the host.

Tolerance of the sums: any order of N products is within N 2^-53 of the sum of
their magnitudes; 4 N 2^-53 also covers the products' own rounding.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drive", [False, True])
@pytest.mark.parametrize("N", [1, 63, 256, 257, 1025, 9000])
def test_first_half_and_kinetic(N, drive):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import _lib as L
    lib = L.load()
    g = np.random.Generator(np.random.PCG64(N))
    dev = lambda *shape: torch.as_tensor(g.standard_normal(shape), device="cuda")
    pos, vel, F, Wi, W = dev(3, N), dev(3, N), dev(3, N), dev(9, N), dev(6)
    ref = pos + 0.1 * dev(3, N)
    mass = dev(N).abs() + 20.0
    im, dt = 1.0 / mass, 0.7
    fe = (ctypes.c_double * 3)(1e-2, -2e-2, 5e-3) if drive else None
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: None if t is None else ctypes.c_void_p(t.data_ptr())
    kick = lambda v: (N, p(v), p(F), p(Wi) if drive else None, p(W) if drive else None, fe, p(im), 0.5 * dt)
    want_p, want_v, want_d = pos.clone(), vel.clone(), torch.full((1,), 7.0, dtype=torch.float64, device="cuda")
    assert lib.mt_md_kick(*kick(want_v), st) == 0
    assert lib.mt_md_drift(N, p(want_p), p(want_v), dt, st) == 0
    assert lib.mt_md_max_disp(N, p(want_p), p(ref), p(want_d), st) == 0
    for check in (ref, None):
        got_p, got_v, d = pos.clone(), vel.clone(), torch.full_like(want_d, 7.0)
        assert lib.mt_md_first_half(*kick(got_v), p(got_p), dt, p(check), p(d) if check is not None else None, st) == 0
        assert torch.equal(got_p, want_p) and torch.equal(got_v, want_v)
        assert torch.equal(d, want_d) == (check is not None)
    assert lib.mt_md_first_half(*kick(got_v), p(got_p), dt, p(ref), None, st) != 0
    out = torch.empty(4, dtype=torch.float64, device="cuda")
    assert lib.mt_md_kinetic(N, p(vel), p(mass), p(out), st) == 0
    v, m, out = vel.cpu().numpy(), mass.cpu().numpy(), out.cpu().numpy()
    terms = [(m * v * v).ravel(), m * v[0], m * v[1], m * v[2]]
    for k, t in enumerate(terms):
        assert abs(out[k] - t.sum()) <= 4 * N * 2.0 ** -53 * np.abs(t).sum(), k
