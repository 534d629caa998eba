"""The batch executor's coefficient tables where the caller's allocator refuses
memory for them: the results keep their bits, a refused size is not asked for
again (every request waits for the stream), an exact fit is tried where there
is no room to grow into, and the table that there was is kept."""
import pytest
import torch

from synth import water_cluster
from tests.gpu_util import say, gpu_params

pytestmark = pytest.mark.gpu

SITES = 100                     # 20 waters
TABLE = SITES * SITES * 16      # FP64 pairs reserved for each cluster


@pytest.fixture
def executor(monkeypatch):
    """An executor whose allocator refuses requests above limit[0] and records
    (bytes, granted) of each, and an unlimited one."""
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2201_00804_amd import batch, _lib
    from paper_2201_00804_amd.engine import TorchAllocator
    limit, asked = [0], []

    class Limited(TorchAllocator):
        def __init__(self, device, stream):
            super().__init__(device, stream)
            grant = self.alloc_fn

            def alloc(nbytes, user):
                asked.append((nbytes, nbytes <= limit[0]))
                return grant(nbytes, user) if nbytes <= limit[0] else None
            self.inner, self.alloc_fn = grant, _lib.ALLOC_FN(alloc)

    free = batch.ClusterBatch(0)
    monkeypatch.setattr(batch, "TorchAllocator", Limited)
    b = batch.ClusterBatch(0)
    yield b, free, limit, asked
    b.close()
    free.close()


def _run(b, count):
    from paper_2201_00804_amd.batch import concat_clusters
    distinct = [water_cluster(20, 3), water_cluster(20, 4), water_cluster(20, 5)]
    off, t = concat_clusters([distinct[k % 3] for k in range(count)], "cuda")
    r = b.run(off, t["xyz"], t["mol"], t["q"], t["dip"], t["quad"], t["alpha"],
              gpu_params(distinct[0], tol=1e-9))
    r.wait()
    return r


def _same(b, free, count):
    r, ref = _run(b, count), _run(free, count)
    assert int(r.status.abs().max()) == 0
    for key in ("mu", "forces", "e_pol", "e_elec", "iters"):
        assert torch.equal(getattr(r, key), getattr(ref, key)), key


def test_refused_table_is_asked_for_once(executor):
    b, free, limit, asked = executor
    limit[0] = 2_000_000
    _same(b, free, 40)                       # 6.4 MB of tables
    say(f"[batch memory] first call asked for {asked}")
    assert any(n >= 40 * TABLE and not ok for n, ok in asked)
    del asked[:]
    _same(b, free, 40)
    assert asked == []
    _same(b, free, 5)                        # fits
    assert asked == [(5 * TABLE, True)]
    del asked[:]
    _same(b, free, 40)                       # five of them have a table now
    assert asked == []


def test_exact_size_and_old_table(executor):
    b, free, limit, asked = executor
    limit[0] = 20 * TABLE - 1
    _same(b, free, 10)
    del asked[:]
    _same(b, free, 15)                       # twice the old size is refused
    say(f"[batch memory] growing asked for {asked}")
    tables = [(n, ok) for n, ok in asked if n % TABLE == 0]
    assert tables == [(20 * TABLE, False), (15 * TABLE, True)]
    del asked[:]
    _same(b, free, 40)
    tables = [(n, ok) for n, ok in asked if n % TABLE == 0]
    assert tables[0] == (40 * TABLE, False) and tables[-1] == (15 * TABLE, True)
    del asked[:]
    _same(b, free, 15)
    _same(b, free, 40)
    assert asked == []
