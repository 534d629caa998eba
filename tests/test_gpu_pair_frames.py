"""Forces with local frames at the list lengths where the FP64 pair loop goes
wrong first: 0, 5, 15, 20, 30, 35 and 195 entries for 16 lanes, one and two
records in turn, and boxes.  The field and gradient that the rotations need come
from the loop's sums without the virial and from pair terms with it; both add up
the same pairs: n 2^-53 of the largest, where the nearest pairs' terms are up to
a thousand times a site's force."""
import numpy as np
import pytest
import torch

from synth import water_cluster, water_box_ortho, water_frames
from tests.gpu_util import say, rel_err
from tests.test_gpu_frames import _engine

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _compare(d, name, **kw):
    say(f"[pair frames] {name}")
    eng = _engine(d, dict(tol=1e-10, **kw), "fp64", water_frames(d))
    eng.solve()
    f = eng.energy_forces()[2].cpu().numpy()
    g = eng.energy_forces(virial=True)[2].cpu().numpy()
    assert np.all(np.isfinite(f))
    assert rel_err(f, g) < 1e-10
    eng.close()


@pytest.mark.parametrize("waters", [1, 2, 4, 5, 7, 8, 40])
def test_cluster_forces(waters):
    _compare(water_cluster(waters, 5), f"cluster {waters}")


@pytest.mark.parametrize("counts", [(3, 3, 4), (6, 5, 7)])
def test_box_forces(counts):
    _compare(water_box_ortho(counts, (3.105,) * 3, 5), f"box {counts}", beta=0.5, cutoff=4.5,
             grid=24)
