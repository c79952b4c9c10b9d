"""GPU: the buffers that a table keeps of its last exploration: the next one
brings no more, a rebuild gives them back, and what they hold of one
exploration does not reach another.  Device memory is read from the driver."""
import pytest

torch = pytest.importorskip("torch")

from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("kind,fused", [("bucketed", False), ("bucketed", True), ("cuckoo", False), ("cuckoo", True)])
def test_kept_buffers(kind, fused):
    model = inputs.BfsModel(1)
    with b.Table(kind, capacity=26 << 20, nhash=4) as t:
        small = t.bfs_explore(model, 3, fused=fused)
        t.clear()
        first = free_bytes()
        r = t.bfs_explore(model, 6, fused=fused)
        kept = free_bytes()
        assert first - kept > 16 * MIB
        if kind == "bucketed":                 # a Cuckoo table's scratch for its batches stays too
            assert first - kept < 1032 * MIB
        t.clear()
        again = t.bfs_explore(model, 6, fused=fused)
        assert kept - free_bytes() < 8 * MIB   # the runtime's own pools grow by 2 MiB now and then
        assert again["batch_sizes"] == r["batch_sizes"] and again["new_counts"] == r["new_counts"]
        size, spare = t.size(), free_bytes()
        t.rebuild()
        assert free_bytes() - spare > 8 * MIB and t.size() == size
        t.clear()
        r = t.bfs_explore(model, 3, fused=fused)
        assert r["batch_sizes"] == small["batch_sizes"] and r["new_counts"] == small["new_counts"]
