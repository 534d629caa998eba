"""Batched clusters at the sizes where the executor changes its path: the
largest small cluster and the smallest large one (60 and 65 sites), the last
size whose coefficient table fits the small path's LDS and the first that
does not (40 and 45 polarizable sites), one and two rows of T per slot of the
large solve (48 and 51 polarizable sites), and the largest solve (640 sites,
all polarizable).  FP64 against the oracle's direct sums, with the bars of the
other batch tests: both solves stop at 1e-10 D, so dipoles agree to 1e-7 of
their largest entry, energies to 1e-9 and forces to 1e-7 (relative RMS).
Every cluster is also bit-identical alone and inside the batch, where small
clusters run beside the large solves."""
import numpy as np
import pytest
import torch

import oracle
from oracle.model import System, Params
from synth import water_cluster
from tests.gpu_util import say, gpu_params, rel_err, rms_rel, pol_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _all_polarizable(d):
    """Every site polarizable, with a fifth of the water model's alpha (the
    barycentres lie 0.48 A from their atoms)."""
    d = dict(d)
    alpha = np.array(d["alpha"], float)
    rows = np.flatnonzero(np.any(alpha != 0, axis=1))
    d["alpha"] = 0.2 * alpha[rows[np.arange(len(alpha)) % len(rows)]]
    return d


CASES = [(12, False), (13, False), (8, True), (9, True), (16, False), (17, False), (128, True)]


def _run(b, systems, prm):
    from paper_2201_00804_amd.batch import concat_clusters
    off, t = concat_clusters(systems, "cuda")
    r = b.run(off, t["xyz"], t["mol"], t["q"], t["dip"], t["quad"], t["alpha"], prm)
    r.wait()
    return r


def test_edges_match_oracle_and_are_independent():
    from paper_2201_00804_amd.batch import ClusterBatch
    systems = [_all_polarizable(water_cluster(w, 30 + k)) if full else water_cluster(w, 30 + k)
               for k, (w, full) in enumerate(CASES)]
    prm = gpu_params(systems[0], tol=1e-10)
    b = ClusterBatch(0)
    res = _run(b, systems, prm)
    for c, s in enumerate(systems):
        ref = oracle.evaluate(System.from_dict(s), Params(method="direct", tol=1e-10))
        r = res.cluster(c)
        rows = pol_rows(s)
        say(f"[batch edges] {len(s['pos'])} sites, {len(rows)} polarizable: "
            f"iters {r['iterations']}/{ref['iters']}")
        assert r["status"] == 0 and abs(r["iterations"] - ref["iters"]) <= 1
        assert rel_err(r["mu"].numpy()[rows], ref["mu"]) < 1e-7
        assert r["e_pol"] == pytest.approx(ref["E_pol"], rel=1e-9)
        assert r["e_elec"] == pytest.approx(ref["E_elec"], rel=1e-9)
        assert rms_rel(r["forces"].numpy(), ref["forces"]) < 1e-7
        alone = _run(b, [s], prm)
        a0, a1 = res.offsets[c], res.offsets[c + 1]
        assert torch.equal(res.mu[a0:a1], alone.mu)
        assert torch.equal(res.forces[a0:a1], alone.forces)
        assert torch.equal(res.e_pol[c:c + 1], alone.e_pol)
        assert torch.equal(res.e_elec[c:c + 1], alone.e_elec)
    b.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_table_bound_changes_nothing(precision):
    """More large clusters than the bounded coefficient tables hold: those
    past the bound re-evaluate their coefficients, with the same bits."""
    from paper_2201_00804_amd.batch import ClusterBatch
    s = water_cluster(200, 3)                    # 1,000 sites: 640^2 table entries reserved
    prm = gpu_params(s, tol=1e-8, precision=precision)
    b = ClusterBatch(0)
    res = _run(b, [s] * 90, prm)                 # 90 * 6.5 MB (FP64) > 512 MB
    assert int(res.status.abs().max()) == 0
    n = len(s["pos"])
    for c in (1, 40, 88, 89):
        assert torch.equal(res.mu[c * n:(c + 1) * n], res.mu[:n])
        assert torch.equal(res.forces[c * n:(c + 1) * n], res.forces[:n])
    assert torch.equal(res.e_pol, res.e_pol[:1].expand(90))
    b.close()
