"""The one-launch solver step (diagonal preconditioner, up to 1,024 polarizable
sites) in mixed precision, at the edges of its wavefronts, partial sums, passes
and range: it also writes the FP32 copy of the direction, takes the replacement
threshold from the device in a cold start, and ends the first run early there.
Against a conjugate gradient in numpy with the FP64 operator on the mixed
engine's own permanent field: both stop at an FP64 residual of 1e-9 D of dipoles
of about 0.5 D (1e-7 of the largest); a replaced residual costs the mixed solve a
few iterations, at most three here."""
import numpy as np
import pytest
import torch

from synth import water_box_ortho, water_cluster
from tests.gpu_util import say, gpu_params, engine_for, pol_rows, rel_err

pytestmark = pytest.mark.gpu

DEBYE = 4.803204
TOL = 1e-9


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _pcg(T, al, E):
    M = lambda v: np.matmul(al, v[:, :, None])[:, :, 0]
    x = M(E)
    r = E - T(x)
    z = M(r)
    p, rz = z.copy(), np.sum(r * z)
    for it in range(100):
        if np.sqrt(np.sum(z * z) / len(E)) * DEBYE <= TOL:
            return x, it
        q = T(p)
        g = rz / np.sum(p * q)
        x, r = x + g * p, r - g * q
        z = M(r)
        old, rz = rz, np.sum(r * z)
        p = z + rz / old * p
    raise AssertionError("no convergence")


def _compare(d, name, **kw):
    say(f"[step mixed] {name}")
    rows, n = pol_rows(d), len(d["pos"])
    al = np.asarray(d["alpha"])[rows][:, [0, 1, 2, 1, 3, 4, 2, 4, 5]].reshape(-1, 3, 3)
    op = engine_for(d, gpu_params(d, tol=TOL, **kw))
    eng = engine_for(d, gpu_params(d, tol=TOL, precision="mixed", **kw))

    def T(v):
        full = np.zeros((n, 3))
        full[rows] = v
        return op.apply_T(torch.as_tensor(full, device="cuda")).cpu().numpy()[rows]

    x, its = _pcg(T, al, eng.permanent_field().cpu().numpy()[rows])
    for _ in range(2):   # the second solve's batches are sized by the first
        mu, it, rms = eng.solve()
        assert rms <= TOL and its - 1 <= it <= its + 3, (it, its)
        assert rel_err(mu.cpu().numpy()[rows], x) < 1e-7
    mu, it, rms = eng.solve(warm_start=True)
    assert rms <= TOL and it <= 1
    assert rel_err(mu.cpu().numpy()[rows], x) < 1e-7
    eng.close()
    op.close()


@pytest.mark.parametrize("waters", [2, 21, 22, 85, 86, 170, 171, 341, 342])
def test_cluster_solves(waters):
    _compare(water_cluster(waters, 4), f"cluster {waters}")


@pytest.mark.parametrize("counts", [(3, 3, 4), (6, 6, 6), (7, 7, 7)])
def test_box_solves(counts):
    _compare(water_box_ortho(counts, (3.105,) * 3, 4), f"box {counts}", beta=0.5, cutoff=4.6,
             grid=24)
