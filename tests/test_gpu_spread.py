"""Spreading where its bricks and chunks can go wrong: bricks with fewer
sites than one staged chunk (21), exactly around one and two chunks, grids
whose brick edges are the small ones (FP64, sizes divisible by 4), the large
ones, and different per axis, for each spline order.  The permanent field
(all sites, charges to quadrupoles) and T p (polarizable sites, dipoles)
against the oracle's SPME: 1e-9 of the largest entry in FP64 (both sides
FP64); in mixed precision 1e-5 (a few tens of FP32 unit roundoffs of a field
whose parts cancel)."""
import numpy as np
import pytest
import torch

from oracle.model import System, apply_T, permanent_field
from synth import water_box_ortho
from tests.gpu_util import say, gpu_params, oracle_params, engine_for, pol_rows, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("counts,grid,order", [
    ((3, 3, 3), (24, 24, 24), 5),    # edges 4: at most a few sites per brick
    ((3, 3, 4), (12, 12, 16), 5),    # edges 4: up to 21 and more per brick
    ((4, 4, 4), (18, 20, 30), 5),    # edges 6, 4 and 5
    ((4, 4, 4), (10, 10, 10), 5),    # edge 6: two chunks and more
    ((5, 4, 4), (10, 12, 16), 4),
    ((4, 5, 4), (12, 18, 20), 6),
])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_spread_edges(counts, grid, order, precision):
    say(f"[spread] {counts} grid {grid} order {order} {precision}")
    d = water_box_ortho(counts, (3.105,) * 3, 11)
    kw = dict(beta=0.5, cutoff=4.5, grid=grid, order=order)
    eng = engine_for(d, gpu_params(d, precision=precision, **kw))
    rows = pol_rows(d)
    s, prm = System.from_dict(d), oracle_params(d, **kw)
    tol = 1e-9 if precision == "fp64" else 1e-5
    assert rel_err(eng.permanent_field().cpu().numpy()[rows], permanent_field(s, prm)) < tol
    p = np.random.default_rng(3).standard_normal((len(d["pos"]), 3))
    tp = eng.apply_T(torch.as_tensor(p, device="cuda")).cpu().numpy()[rows]
    assert rel_err(tp, apply_T(s, prm, p[rows])) < tol
    eng.close()
