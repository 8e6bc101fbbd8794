"""The displacement check with atoms whose displacement is not a number: the maximum
over the others, as with fmax, wherever in a wavefront or block they are; an
infinite displacement is the maximum.
"""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("N", [64, 257, 1000])
def test_not_a_number_among_displacements(N, fused):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import _lib as L
    lib = L.load()
    g = np.random.Generator(np.random.PCG64(N))
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    dev = lambda a: torch.as_tensor(a, device="cuda")
    zero, one = dev(np.zeros((3, N))), dev(np.ones(N))
    ref = g.standard_normal((3, N))
    moved = ref + g.standard_normal((3, N))
    out = torch.empty(1, dtype=torch.float64, device="cuda")

    def check(pos):
        r, q = dev(ref), dev(pos)
        if fused:
            v = zero.clone()
            rc = lib.mt_md_first_half(N, p(v), p(zero), None, None, None, p(one), 0.5, p(q), 0.5, p(r), p(out), st)
        else:
            rc = lib.mt_md_max_disp(N, p(q), p(r), p(out), st)
        assert rc == 0
        return float(out.cpu()[0])

    for bad in (0, 1, 31, 62, 63, N // 2, N - 1):
        for value in (np.nan, -np.nan):
            pos = moved.copy()
            pos[1, bad] = value
            d2 = ((pos - ref) ** 2).sum(0)
            want = np.nanmax(d2)
            assert abs(check(pos) - want) <= 1e-15 * want, (bad, value)
    pos = moved.copy()
    pos[0, N // 3] = -np.inf
    assert check(pos) == np.inf
    assert check(np.full((3, N), np.nan)) == 0.0
