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
