"""Spreading bricks at their edges.

One brick that holds exactly one and two staged chunks of sites (21 each) and
one site fewer or more, all within each other's reach, so that every grid point
of the brick is added to by one site after the other: 24^3 points at order 5 are
cut into bricks of 4^3 in FP64 and 8^3 in mixed precision, and the sites have
their base points in the first 4 of each axis.

Axes cut into bricks of unequal length (FP64): at order 6 into K / 5 of them, at
least order - 1 = 5 points long (16: 6, 5, 5; 32: 6, 5, 5, 6, 5, 5; 36: 6 and six
of 5), at order 4 into K / 4 (18: 5, 4, 5, 4; 30: seven of 5 and 4), and at order
5 again 18 and 30.

The permanent field (all sites, charges to quadrupoles) and T p (dipoles) against
the oracle's SPME on the same grid: 1e-9 of the largest entry in FP64 on both
sides, 1e-5 in mixed precision (a few tens of FP32 unit roundoffs of a field
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


def _compare(d, precision, **kw):
    eng = engine_for(d, gpu_params(d, precision=precision, **kw))
    rows = pol_rows(d)
    s, prm = System.from_dict(d), oracle_params(d, **kw)
    tol = 1e-9 if precision == "fp64" else 1e-5
    assert rel_err(eng.permanent_field().cpu().numpy()[rows], permanent_field(s, prm)) < tol
    p = np.random.default_rng(3).standard_normal((len(d["pos"]), 3))
    tp = eng.apply_T(torch.as_tensor(p, device="cuda")).cpu().numpy()[rows]
    assert rel_err(tp, apply_T(s, prm, p[rows])) < tol
    eng.close()


def _one_brick(n):
    """n sites of their own molecules on a jittered lattice in [0, 4)^3, in a
    box of 24 A."""
    d = dict(water_box_ortho((3, 3, 3), (8.0,) * 3, 5))
    rng = np.random.default_rng(n)
    at = np.stack(np.meshgrid(*[np.arange(4)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pos = rng.permutation(at)[:n] + 0.5 + rng.uniform(-0.2, 0.2, (n, 3))
    assert np.all(np.floor(pos) >= 0) and np.all(np.floor(pos) < 4)
    pol = pol_rows(d)
    for k in ("q", "dip", "quad"):
        d[k] = np.asarray(d[k])[:n]
    d["alpha"] = np.asarray(d["alpha"])[pol[:n]]
    d.update(pos=pos, mol=np.arange(n, dtype=np.int32), box=np.array([24.0, 24.0, 24.0]))
    return d


@pytest.mark.parametrize("sites", [20, 21, 22, 42, 43, 64])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_chunks_of_one_brick(sites, precision):
    say(f"[spread bricks] {sites} sites {precision}")
    _compare(_one_brick(sites), precision, beta=0.5, cutoff=4.5, grid=(24, 24, 24), order=5)


@pytest.mark.parametrize("grid,order", [
    ((16, 32, 36), 6), ((36, 16, 32), 6), ((18, 30, 16), 4), ((18, 30, 20), 5)])
def test_unequal_bricks(grid, order):
    say(f"[spread bricks] grid {grid} order {order}")
    d = water_box_ortho((4, 4, 5), (3.105,) * 3, 11)
    _compare(d, "fp64", beta=0.5, cutoff=4.5, grid=grid, order=order)
