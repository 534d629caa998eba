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


@pytest.mark.parametrize("grid", [(64, 64, 16), (64, 72, 16), (16, 10, 18)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fold_in_the_plane_pass(monkeypatch, grid, precision):
    """Planes up to and past the largest that sum the spreading tiles in the
    first pass of the convolution, against the five-pass convolution, which
    never does (the same sums and another order of the transforms: rounding,
    1e-12 of FP64 and 1e-5 of FP32)."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    say(f"[gather] fold grid {grid} {precision}")
    d = water_box_ortho((3, 4, 4), (3.105,) * 3, 13)
    p = torch.as_tensor(np.random.default_rng(4).standard_normal((len(d["pos"]), 3)), device="cuda")
    out = []
    for planes in ("1", "0"):
        monkeypatch.setenv("SIBFA_FFT_PLANES", planes)
        eng = engine_for(d, gpu_params(d, precision=precision, beta=0.5, cutoff=4.5, grid=grid))
        out.append((eng.permanent_field().cpu().numpy(), eng.apply_T(p).cpu().numpy()))
        eng.close()
    tol = 1e-12 if precision == "fp64" else 1e-5
    assert rel_err(out[0][0], out[1][0]) < tol and rel_err(out[0][1], out[1][1]) < tol
