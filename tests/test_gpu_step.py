"""The solver's update, stop test and direction in one workgroup (diagonal
preconditioner, up to 1,024 polarizable sites) at the edges of its wavefronts,
partial sums, passes and range, against the same conjugate gradient written in
numpy around the engine's operator.  Both stop at an RMS change of 1e-9 D of
dipoles of about 0.5 D and differ by rounding before that: dipoles within 1e-7
of the largest, iteration counts within one."""
import numpy as np
import pytest
import torch

from synth import water_box_ortho, water_cluster
from tests.gpu_util import say, gpu_params, engine_for, pol_rows, rel_err

pytestmark = pytest.mark.gpu

DEBYE = 4.803204


def _pcg(eng, d, tol):
    rows = pol_rows(d)
    a6 = np.asarray(d["alpha"])[rows]
    al = a6[:, [0, 1, 2, 1, 3, 4, 2, 4, 5]].reshape(-1, 3, 3)
    n = len(d["pos"])

    def T(v):
        full = np.zeros((n, 3))
        full[rows] = v
        return eng.apply_T(torch.as_tensor(full, device="cuda")).cpu().numpy()[rows]

    def M(v):
        return np.matmul(al, v[:, :, None])[:, :, 0]

    E = eng.permanent_field().cpu().numpy()[rows]
    x = M(E)
    r = E - T(x)
    z = M(r)
    p, rz = z.copy(), np.sum(r * z)
    for it in range(100):
        if np.sqrt(np.sum(z * z) / len(rows)) * DEBYE <= tol:
            return x, it
        q = T(p)
        g = rz / np.sum(p * q)
        x, r = x + g * p, r - g * q
        z = M(r)
        old, rz = rz, np.sum(r * z)
        p = z + rz / old * p
    raise AssertionError("no convergence")


@pytest.mark.parametrize("waters", [2, 21, 22, 85, 86, 170, 171, 341, 342])
def test_cluster_solves(waters):
    _compare(water_cluster(waters, 4), f"cluster {waters}")


@pytest.mark.parametrize("counts", [(3, 3, 4), (6, 6, 6), (7, 7, 7)])
def test_box_solves(counts):
    _compare(water_box_ortho(counts, (3.105,) * 3, 4), f"box {counts}", beta=0.5, cutoff=4.6,
             grid=24)


def _compare(d, name, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    say(f"[step] {name}")
    eng = engine_for(d, gpu_params(d, tol=1e-9, **kw))
    x, n = _pcg(eng, d, 1e-9)
    for _ in range(2):   # the second solve's batches are sized by the first
        mu, it, rms = eng.solve()
        assert rms <= 1e-9 and abs(it - n) <= 1, (it, n)
        assert rel_err(mu.cpu().numpy()[pol_rows(d)], x) < 1e-7
    eng.close()
