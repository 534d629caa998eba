"""Offsets on the device whose difference overflows an int: the ranges are
reported as invalid (the difference of the two extremes wraps to 1) and the
clusters with valid ones are evaluated."""
import math

import pytest
import torch

from synth import water_cluster
from tests.gpu_util import say, gpu_params
from tests.test_zz_no_alloc import _noalloc, _outputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waters", [3, 20])
def test_wrapping_ranges_are_reported(waters):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2201_00804_amd import _lib
    from paper_2201_00804_amd.batch import concat_clusters
    s = water_cluster(waters, 5)
    off, t = concat_clusters([s], "cuda")
    n, top, low = off[-1], 2 ** 31 - 1, -2 ** 31
    say(f"[batch ranges] {n} sites")
    ranges = torch.as_tensor([0, n, top, low, n, 0, n], dtype=torch.int32, device="cuda")
    out = _outputs(n, 6, "cuda")
    assert _noalloc(_lib.load(), ranges, n, t, gpu_params(s, tol=1e-9), out,
                    torch.cuda.current_stream()) == 0
    torch.cuda.synchronize()
    assert out["status"].tolist() == [0, -1, -1, -1, -1, 0]
    e = out["e_pol"].tolist()
    assert e[0] == e[5] and e[0] < 0 and all(math.isnan(x) for x in e[1:5])
