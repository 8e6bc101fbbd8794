"""The launch shapes that mt_autotune times: fixed candidate tiles and the open tile
(tile=0) that untuned calls use.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_open_tile_is_a_candidate(tmp_path, precision):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_11474_amd import api
    g = np.random.Generator(np.random.PCG64(1))
    s = W.make_set(W.strained_diamond_cells(2, 3) + [W.random_packing(g, 40)])
    ts = api.from_structures(s)
    X = W.draw_params(g, 7)
    ref = ts.tersoff_eval(W.draw_params(g, 1), precision="fp64")
    n = torch.as_tensor(s.sizes(), dtype=torch.float64, device="cuda")
    ts.attach_reference(ref["E"][0] / n, ref["W"][0] / n[:, None], ref["F"][0])
    want = ts.fitness(X, precision=precision).clone()
    path = tmp_path / "shapes"
    ts.autotune(len(X), precision, str(path))
    lines = path.read_text().splitlines()
    field = lambda line, k: float(line.split(k + "=")[1].split()[0])
    timed = [l for l in lines if l.startswith("#") and "burst_ms" not in l]
    assert {field(l, "block") for l in timed if " tile=0 " in l} == {field(l, "block") for l in timed}
    chosen = [l for l in lines if not l.startswith("#")]
    assert len(chosen) == 1 and field(chosen[0], " ms") <= min(field(l, " ms") for l in timed) * (1 + 1e-4)
    assert torch.equal(ts.fitness(X, precision=precision), want)
    ts.close()
