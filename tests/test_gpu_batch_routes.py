"""Where a batch's small clusters run: in a launch of their own (no large
cluster, or more clusters than the large solves leave CUs for) or beside the
large solves; chosen on the host, and on the device where the offsets are there
only.  Every route gives a cluster the bits it has alone."""
import numpy as np
import pytest
import torch

from synth import water_cluster
from tests.gpu_util import say, gpu_params
from tests.test_zz_no_alloc import _noalloc, _outputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def _systems(counts):
    """Clusters of counts = {waters: number} in a fixed shuffled order."""
    sizes = np.repeat(list(counts), list(counts.values()))
    np.random.default_rng(2).shuffle(sizes)
    distinct = {w: [water_cluster(int(w), 20 + w), water_cluster(int(w), 120 + w)]
                for w in counts}
    return [distinct[w][k % 2] for k, w in enumerate(sizes)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("counts", [
    {2: 5, 12: 4},          # no large cluster, more sites than one small cluster
    {2: 900, 13: 4},        # apart: the small clusters would take longer than the solves
    {2: 270, 64: 2},        # beside: the solves take longer
    {4: 3, 20: 3},          # beside: fewer clusters than CUs
])
def test_routes_keep_the_bits(counts, precision):
    from paper_2201_00804_amd import _lib
    from paper_2201_00804_amd.batch import ClusterBatch, concat_clusters
    say(f"[batch routes] {counts} {precision}")
    systems = _systems(counts)
    prm = gpu_params(systems[0], tol=1e-9, precision=precision)
    off, t = concat_clusters(systems, "cuda")
    n, nc = off[-1], len(systems)
    b = ClusterBatch(0)

    def run(off, t):
        r = b.run(off, t["xyz"], t["mol"], t["q"], t["dip"], t["quad"], t["alpha"], prm)
        r.wait()
        return r

    ref = run(off, t)
    out = _outputs(n, nc, "cuda")
    off_dev = torch.as_tensor(off, dtype=torch.int32, device="cuda")
    assert _noalloc(_lib.load(), off_dev, n, t, prm, out, torch.cuda.current_stream()) == 0
    torch.cuda.synchronize()
    for key in ("mu", "forces", "e_pol", "e_elec", "iters", "rms", "status"):
        assert torch.equal(out[key], getattr(ref, key)), key
    assert int(ref.status.abs().max()) == 0
    seen = set()
    for c, s in enumerate(systems):
        if id(s) in seen:
            continue
        seen.add(id(s))
        alone = run(*concat_clusters([s], "cuda"))
        assert torch.equal(ref.mu[off[c]:off[c + 1]], alone.mu)
        assert torch.equal(ref.forces[off[c]:off[c + 1]], alone.forces)
        assert torch.equal(ref.e_pol[c:c + 1], alone.e_pol)
    b.close()


def test_overlapping_ranges_are_all_solved():
    """Offsets on the device that name one large cluster several times: more
    large clusters than the sites could hold side by side."""
    from paper_2201_00804_amd import _lib
    from paper_2201_00804_amd.batch import concat_clusters
    s = water_cluster(20, 7)
    off, t = concat_clusters([s], "cuda")
    n = off[-1]
    prm = gpu_params(s, tol=1e-9)
    ranges = torch.as_tensor([0, n, 0, n, 0, n, 0, n], dtype=torch.int32, device="cuda")
    out = _outputs(n, 7, "cuda")
    one = _outputs(n, 1, "cuda")
    lib, st = _lib.load(), torch.cuda.current_stream()
    assert _noalloc(lib, ranges, n, t, prm, out, st) == 0
    assert _noalloc(lib, ranges[:2].contiguous(), n, t, prm, one, st) == 0
    torch.cuda.synchronize()
    assert out["status"].tolist() == [0, -1, 0, -1, 0, -1, 0]
    assert torch.equal(out["mu"], one["mu"]) and torch.equal(out["forces"], one["forces"])
    assert torch.equal(out["e_pol"][::2], one["e_pol"].expand(4))


@pytest.mark.parametrize("counts", [{2: 5}, {2: 900, 13: 4}, {2: 270, 64: 2}])
def test_routes_under_capture(counts):
    """The call without an executor recorded into a graph, on each route, and
    replayed between other work on new positions: the eager call's bits."""
    from paper_2201_00804_amd import _lib
    from paper_2201_00804_amd.batch import concat_clusters
    lib, systems = _lib.load(), _systems(counts)
    prm = gpu_params(systems[0], tol=1e-9)
    off, t = concat_clusters(systems, "cuda")
    n, nc = off[-1], len(systems)
    off_dev = torch.as_tensor(off, dtype=torch.int32, device="cuda")
    out, ref = _outputs(n, nc, "cuda"), _outputs(n, nc, "cuda")
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        assert _noalloc(lib, off_dev, n, t, prm, out, st) == 0
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        assert _noalloc(lib, off_dev, n, t, prm, out, torch.cuda.current_stream()) == 0
    rng = np.random.default_rng(4)
    for k in range(3):
        t["xyz"] += torch.as_tensor(rng.uniform(-0.01, 0.01, (n, 3)), device="cuda")
        graph.replay()
        torch.cuda.synchronize()
        # the eager call shares the scratch: only after the replay
        assert _noalloc(lib, off_dev, n, t, prm, ref, torch.cuda.current_stream()) == 0
        torch.cuda.synchronize()
        say(f"[batch routes] replay {k} of {nc} clusters")
        for key in ("mu", "forces", "e_pol", "e_elec", "iters", "status"):
            assert torch.equal(out[key], ref[key]), key
        assert int(out["status"].abs().max()) == 0
