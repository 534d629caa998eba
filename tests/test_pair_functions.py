"""The FP64 functions of the pair loops (csrc/erfcx_fit.h: erfcx as powers of u,
exp(r) = 1 + r + r^2 q(r)), evaluated on the host in the kernels' steps, and
on the GPU the forces from summed potentials against the pair forces that the
virial needs."""
import os
import re

import numpy as np
import pytest
import torch
from scipy.special import erfcx

HEADER = os.path.join(os.path.dirname(os.path.abspath(__file__)), os.pardir,
                      "paper_2201_00804_amd", "csrc", "erfcx_fit.h")


def _array(name):
    body = re.search(rf"{name}\[\d+\] = \{{(.*?)\}};", open(HEADER).read(), re.S).group(1)
    return [float(v) for v in body.replace(",", " ").split()]


def _horner(c, x):
    y = np.full_like(x, c[-1])
    for v in c[-2::-1]:
        y = y * x + v
    return y


def test_erfcx_powers():
    """Same bound as the Chebyshev form's test."""
    t0 = 1.0 / 2.2
    x = np.linspace(0.0, 6.0, 200001)
    u = (1.0 / (1.0 + 0.2 * x) - t0) * (2.0 / (1.0 - t0)) - 1.0
    assert np.abs(_horner(_array("kErfcxMF64"), u) / erfcx(x) - 1.0).max() < 3e-14


def test_exp():
    """Rounding of the reduced argument (|k| ln 2 in two parts: 2^-54 |r|) and
    of the last two sums: 2 units of 2^-52."""
    x = -np.concatenate([np.linspace(0.0, 50.0, 200001), np.linspace(50.0, 690.0, 50001)])
    k = np.rint(x * 1.4426950408889634)
    r = (x.astype(np.longdouble) - k * np.longdouble(0.6931471805599453)).astype(np.float64)
    r = r - k * 2.3190468138462996e-17
    e = np.ldexp((r * r * _horner(_array("kExpQ"), r) + r) + 1.0, k.astype(int))
    ref = np.exp(x.astype(np.longdouble))
    assert float(np.abs(e / ref - 1).max()) < 4.5e-16


@pytest.mark.gpu
@pytest.mark.parametrize("waters", [1, 2, 4, 5, 7, 8, 40])
@pytest.mark.parametrize("thole", [None, (0.2, 0.6)])
def test_cluster_forces(waters, thole):
    """Lists of 0, 5, 15, 20, 30, 35 and 195 entries for 16 lanes, one and two
    records in turn."""
    from synth import water_cluster
    _compare(water_cluster(waters, 5), thole, f"cluster {waters}")


@pytest.mark.gpu
@pytest.mark.parametrize("counts", [(3, 3, 4), (6, 5, 7)])
@pytest.mark.parametrize("thole", [None, (0.2, 0.6)])
def test_box_forces(counts, thole):
    from synth import water_box_ortho
    _compare(water_box_ortho(counts, (3.105,) * 3, 5), thole, f"box {counts}",
             beta=0.5, cutoff=4.5, grid=24)


def _compare(d, thole, name, **kw):
    """Sums of n terms of the same pairs: n 2^-53 of the largest, and the
    nearest pairs' terms are up to a thousand times a site's force."""
    from tests.gpu_util import say, gpu_params, engine_for, rel_err
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    say(f"[pair forces] {name} thole {thole}")
    if thole:
        rng = np.random.default_rng(2)
        d["thole"] = rng.uniform(*thole, len(d["pos"]))
    eng = engine_for(d, gpu_params(d, tol=1e-10, **kw))
    eng.solve()
    f = eng.energy_forces()[2].cpu().numpy()
    g = eng.energy_forces(virial=True)[2].cpu().numpy()
    assert np.all(np.isfinite(f))
    assert rel_err(f, g) < 1e-10
    eng.close()
