"""Neighbour lists where the builder's split of a cell among wavefronts and
its stencil can go wrong: clusters (one cell) around the 64-candidate chunk
and the 256-site pass, boxes with fewer than five cells along some or all
axes, with exactly five, and with more cells than wavefronts are dealt to;
and the records of cells larger than the sort's passes.
Counts are whole numbers and must be exact; the lists' contents are checked
through the permanent field, within 1e-9 of its largest entry (both sides
FP64: a missing or doubled pair at the cutoff is above 1e-5 of it)."""
import numpy as np
import pytest
import torch
from scipy.spatial import cKDTree

from oracle.model import System, permanent_field
from synth import water_cluster, water_box_ortho
from tests.gpu_util import say, gpu_params, oracle_params, engine_for, pol_rows, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("waters", [1, 12, 13, 51, 52, 70])
def test_cluster_lists(waters):
    say(f"[lists] cluster of {waters}")
    d = water_cluster(waters, 3)
    eng = engine_for(d, gpu_params(d))
    got = eng.neighbor_counts().cpu().numpy()
    assert np.all(got == len(d["pos"]) - 5)
    E = eng.permanent_field().cpu().numpy()[pol_rows(d)]
    ref = permanent_field(System.from_dict(d), oracle_params(d))
    if waters > 1:
        assert rel_err(E, ref) < 1e-9
    eng.close()


@pytest.mark.parametrize("counts,cutoff", [
    ((3, 3, 4), 4.5),      # 4, 4 and 5 cells
    ((4, 4, 4), 6.0),      # 4 cells along every axis
    ((4, 4, 8), 4.9),      # 5, 5 and 10 cells
    ((3, 9, 5), 4.6),      # 4, 12 and 6 cells
    ((14, 13, 15), 5.0),   # more cells than one wavefront per site needs
])
def test_box_lists(counts, cutoff):
    say(f"[lists] box {counts} cutoff {cutoff}")
    d = water_box_ortho(counts, (3.105,) * 3, 7)
    grid = tuple(int(2 * np.ceil(0.6 * b)) for b in d["box"])
    grid = tuple(next(k for k in range(max(g, 10), 200, 2) if not _other_factors(k)) for g in grid)
    kw = dict(beta=0.5, cutoff=cutoff, grid=grid)
    eng = engine_for(d, gpu_params(d, **kw))
    got = eng.neighbor_counts().cpu().numpy()
    box = np.asarray(d["box"])
    tree = cKDTree(np.mod(d["pos"], box), boxsize=box)
    pairs = tree.query_pairs(cutoff, output_type="ndarray")
    pairs = pairs[d["mol"][pairs[:, 0]] != d["mol"][pairs[:, 1]]]
    assert np.array_equal(got, np.bincount(pairs.ravel(), minlength=len(d["pos"])))
    if len(d["pos"]) < 2000:
        E = eng.permanent_field().cpu().numpy()[pol_rows(d)]
        ref = permanent_field(System.from_dict(d), oracle_params(d, **kw))
        assert rel_err(E, ref) < 1e-9
    eng.close()


@pytest.mark.parametrize("counts,spacing", [
    ((4, 4, 4), 3.105),    # a few sites per cell
    ((10, 10, 10), 1.6),   # 78 on average: more than one wavefront pass
    ((15, 15, 15), 1.4),   # 264 on average: beyond the rank sort's buffer
])
def test_cell_records(counts, spacing):
    """A re-sort writes each cell's records and polarizable indices itself;
    new polarizabilities on the same sort go through the scan over all sites.
    Same numbers in, same operations on them: equal bit for bit.  Sites in
    another caller order sort differently within the cells: the same sums to
    rounding (n * 2^-53 of the largest term, below 1e-10)."""
    say(f"[lists] records {counts} spacing {spacing}")
    d = water_box_ortho(counts, (3.105,) * 3, 7)
    d["pos"] = d["pos"] * (spacing / 3.105)   # denser than molecules fit
    d["box"] = d["box"] * (spacing / 3.105)
    n = len(d["pos"])
    rng = np.random.default_rng(5)
    d["alpha"] = d["alpha"] * (rng.random(n) < 0.6)[:, None]
    grid = tuple(next(k for k in range(max(2 * int(0.6 * b), 10), 200, 2) if not _other_factors(k))
                 for b in d["box"])
    cutoff = float(np.min(d["box"])) / 2 * 0.999
    prm = gpu_params(d, beta=0.5, cutoff=cutoff, grid=grid)
    p = torch.as_tensor(rng.standard_normal((n, 3)), device="cuda:0")
    p[torch.as_tensor(~np.any(d["alpha"] != 0, axis=1), device="cuda:0")] = 0
    eng = engine_for(d, prm)
    E1, T1 = eng.permanent_field(), eng.apply_T(p)
    eng.set_polarizabilities(torch.as_tensor(d["alpha"], device="cuda:0").contiguous())
    E2, T2 = eng.permanent_field(), eng.apply_T(p)
    assert torch.equal(E1, E2) and torch.equal(T1, T2)
    eng.close()
    order = rng.permutation(n)
    back = torch.as_tensor(np.argsort(order), device="cuda:0")
    r = {k: (v[order] if getattr(v, "shape", ())[:1] == (n,) else v) for k, v in d.items()}
    eng = engine_for(r, prm)
    E3 = eng.permanent_field()[back]
    T3 = eng.apply_T(p[torch.as_tensor(order, device="cuda:0")].contiguous())[back]
    assert rel_err(E3.cpu(), E1.cpu()) < 1e-10 and rel_err(T3.cpu(), T1.cpu()) < 1e-10
    eng.close()


def _other_factors(k):
    for f in (2, 3, 5):
        while k % f == 0:
            k //= f
    return k != 1
