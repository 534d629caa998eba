"""The gathers from the potential grid on the smallest grids (2 order points
along x, so that most sites' rows run over the grid's edge into the repeated
points), for both convolution paths, which write those points.  Against the
oracle: FP64 1e-9 as everywhere (a wrong grid point is of the order of the
value itself), mixed 1e-5 (the FP32 grid)."""
import numpy as np
import pytest
import torch

import oracle
from oracle.model import System, apply_T, permanent_field
from synth import water_box_ortho
from tests.gpu_util import say, gpu_params, oracle_params, engine_for, pol_rows, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planes", ["1", "0"])
@pytest.mark.parametrize("order,grid", [(4, (8, 10, 12)), (5, (10, 12, 16)), (6, (12, 16, 18))])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_rows_over_the_edge(monkeypatch, planes, order, grid, precision):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    say(f"[gather] order {order} grid {grid} planes {planes} {precision}")
    monkeypatch.setenv("SIBFA_FFT_PLANES", planes)
    d = water_box_ortho((3, 4, 4), (3.105,) * 3, 12)
    kw = dict(beta=0.5, cutoff=4.5, grid=grid, order=order)
    eng = engine_for(d, gpu_params(d, precision=precision, **kw))
    rows = pol_rows(d)
    s, prm = System.from_dict(d), oracle_params(d, **kw)
    tol = 1e-9 if precision == "fp64" else 1e-5
    assert rel_err(eng.permanent_field().cpu().numpy()[rows], permanent_field(s, prm)) < tol
    p = np.random.default_rng(3).standard_normal((len(d["pos"]), 3))
    tp = eng.apply_T(torch.as_tensor(p, device="cuda")).cpu().numpy()[rows]
    assert rel_err(tp, apply_T(s, prm, p[rows])) < tol
    if precision == "fp64":
        eng.solve()
        assert rel_err(eng.energy_forces()[2].cpu().numpy(), oracle.evaluate(s, prm)["forces"]) < 1e-7
    eng.close()
