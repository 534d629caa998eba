"""Field and forces of large clusters at the edges of the site chunks that
their kernels stage (128 sites): one chunk short of a site, full, one site
more, and the same around two.  Clusters of any number of sites are cut from
water clusters.  FP64 against the oracle's direct sums with the bars of the
other batch tests (both solves stop at 1e-10 D: dipoles 1e-7 of the largest,
energies 1e-9, forces 1e-7 relative RMS); in mixed precision the pair terms
are FP32 and summed in FP64: dipoles, E_pol and forces within 1e-4, as for other
mixed batches, and E_elec, whose up to 33,000 terms of some 100 kcal/mol cancel
(1e-6 of each after a dozen roundings, of either sign), within 0.02 kcal/mol."""
import numpy as np
import pytest
import torch

import oracle
from oracle.model import System, Params
from synth import water_cluster
from tests.gpu_util import say, gpu_params, rel_err, rms_rel, pol_rows

pytestmark = pytest.mark.gpu


def _cut(d, n):
    return {k: (v[:n] if isinstance(v, np.ndarray) and len(v) == len(d["pos"]) else v)
            for k, v in d.items()}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_chunk_edges(precision):
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2201_00804_amd.batch import ClusterBatch, concat_clusters
    sizes = [66, 127, 128, 129, 255, 256, 257]
    systems = [_cut(water_cluster((n + 4) // 5, 50 + n), n) for n in sizes]
    prm = gpu_params(systems[0], tol=1e-10, precision=precision)
    b = ClusterBatch(0)
    off, t = concat_clusters(systems, "cuda")
    assert [e - s for s, e in zip(off[:-1], off[1:])] == sizes
    res = b.run(off, t["xyz"], t["mol"], t["q"], t["dip"], t["quad"], t["alpha"], prm)
    for c, s in enumerate(systems):
        ref = oracle.evaluate(System.from_dict(s), Params(method="direct", tol=1e-10))
        r, rows = res.cluster(c), pol_rows(s)
        say(f"[batch stage] {precision} {sizes[c]} sites")
        assert r["status"] == 0
        bar = dict(mu=1e-7, e=1e-9, f=1e-7) if precision == "fp64" else dict(mu=1e-4, e=1e-4, f=1e-4)
        assert rel_err(r["mu"].numpy()[rows], ref["mu"]) < bar["mu"]
        assert r["e_pol"] == pytest.approx(ref["E_pol"], rel=bar["e"])
        assert r["e_elec"] == pytest.approx(ref["E_elec"], rel=1e-9,
                                            abs=0.0 if precision == "fp64" else 0.02)
        assert rms_rel(r["forces"].numpy(), ref["forces"]) < bar["f"]
    b.close()
