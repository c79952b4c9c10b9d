"""GPU: what a served run leaves for later calls on its tables: keys put by
merged requests count, so that a later call of as many is not taken for a
table's first batch, and the run has reserved what its unmerged requests could
need.  Flags against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_flags_r2  # noqa: E402
from test_gpu_reserve import free_bytes, loaded  # noqa: E402,F401
from test_gpu_routes import dev, routes  # noqa: E402

pytestmark = pytest.mark.gpu


def pinned(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).pin_memory()


def test_merged_requests_count_as_puts():
    sizes = ((1 << 18, 1 << 19, "bucketed", "bucketed_fop"), (1000, 2048, "bucketed", "bucketed_fop"),
             (5000, 8192, "cuckoo", "cuckoo_probe"))
    tables = [b.Table(kind, capacity=cap, nhash=4) for _, cap, kind, _ in sizes]
    keys = [inputs.uniform_keys(n, seed=n) for n, _, _, _ in sizes]
    srv = b.Server(tables, merge=16)
    outs = srv.run([("put", i, pinned(k), 0.0) for i, k in enumerate(keys)])[0]
    srv.close()
    for t, k, o, (_, _, _, name) in zip(tables, keys, outs, sizes):
        ref = Oracle()
        check_flags_r2(k, o.numpy(), ref.find_or_put(k), name)
        r = routes(lambda: t.find_or_put(dev(k)))              # as many as it holds: not a first batch
        assert name in r and not {"tile_insert", "tile_whole", "cuckoo_whole"} & set(r), r
        assert t.size() == k.size
        t.close()


def test_a_run_reserves_what_unmerged_requests_need():
    n = 1 << 19
    first, keys = inputs.uniform_keys(n, seed=1), inputs.uniform_keys(n, seed=1, start=n)
    k, out = dev(keys), torch.empty(n, dtype=torch.uint8, device="cuda")
    with b.Table("bucketed", capacity=3 * n, nhash=3, bucket_slots=8) as t:
        srv = b.Server([t], merge=1)
        o = srv.run([("put", 0, pinned(first[:1000]), 0.0), ("put", 0, pinned(first[:900]), 0.0)])[0]
        assert o[0].all() and not o[1].any()
        # the table holds as much as this request brings: direct kernels, and the workspace is there all the same
        t.find_or_put(dev(first))
        b.ht_timing_enable(True)
        o = srv.run([("put", 0, pinned(keys), 0.0)])[0]
        names = set(b.ht_timing_report())
        b.ht_timing_enable(False)
        assert "tile_insert" not in names and o[0].all()
        srv.close()
        t.clear()
        before = free_bytes()
        assert "tile_insert" in routes(lambda: t.find_or_put(k, out))
        assert free_bytes() == before and t.size() == n
