"""GPU: calls within a reservation allocate nothing and take the passes that it
was made for, also where a smaller batch needs more of the workspace than the
reserved one; a call beyond it grows it once.  Device memory is read from the
driver, and the timing report says which kernels ran."""
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_dump_r3  # noqa: E402
from test_gpu_routes import dev, routes  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def loaded():
    """The runtime has loaded the passes and made its events before memory is compared."""
    with b.Table("bucketed", capacity=1 << 23, nhash=3, bucket_slots=8, max_batch=1 << 22) as t:
        for n in (1 << 19, 1 << 22):
            t.clear()
            routes(lambda: t.find_or_put(dev(inputs.uniform_keys(n, seed=n))))


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


# slots, reserved, keys of the calls
CASES = [
    (1 << 22, 1 << 21, ((1 << 21) - 1, 1 << 21, 1 << 20)),      # one key less takes the shorter chunks
    (1 << 22, 1 << 22, (1 << 21, 3 << 20, 1 << 20)),            # more reserved than the table can hold
    (1 << 23, 1 << 27, ((1 << 22) + 4097, (1 << 21) - 4096)),   # more than any tiled batch
    (1 << 20, (1 << 19) + 5, (1 << 19, 1 << 18)),
]


@pytest.mark.parametrize("at_create", [False, True])
@pytest.mark.parametrize("cap,reserved,calls", CASES)
def test_calls_within_a_reservation(cap, reserved, calls, at_create):
    keys = [dev(inputs.uniform_keys(n, seed=n)) for n in calls]
    out = torch.empty(max(calls), dtype=torch.uint8, device="cuda")
    with b.Table("bucketed", capacity=cap, nhash=3, bucket_slots=8, max_batch=reserved if at_create else 0) as t:
        if not at_create:
            b.ht_reserve(t.handle, reserved)
        t.find_or_put(keys[0][:1000], out)
        t.clear()
        for k in keys + keys[::-1]:
            before = free_bytes()              # the checks below make tensors of their own
            r = routes(lambda: t.find_or_put(k, out))
            assert "tile_insert" in r, (cap, reserved, k.numel(), r)
            assert free_bytes() == before, (cap, reserved, k.numel())
            assert out[:k.numel()].all() and t.size() == k.numel()
            t.clear()


def test_calls_beyond_a_reservation_grow_it_once():
    n = 1 << 21
    k, out = dev(inputs.uniform_keys(n, seed=3)), torch.empty(n, dtype=torch.uint8, device="cuda")
    with b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=16, max_batch=1 << 18) as t:
        t.find_or_put(k[:1000], out)
        t.clear()
        first = free_bytes()
        assert "tile_insert" in routes(lambda: t.find_or_put(k, out))
        assert first - free_bytes() >= 11 * n
        for m in (n, n - 1, n // 2):
            t.clear()
            grown = free_bytes()
            assert "tile_insert" in routes(lambda: t.find_or_put(k[:m], out))
            assert free_bytes() == grown and t.size() == m


def test_a_rebuild_keeps_the_reservation():
    n = 1 << 20
    keys = inputs.uniform_keys(n, seed=5)
    k, out = dev(keys), torch.empty(n, dtype=torch.uint8, device="cuda")
    for reserved in (0, n):
        with b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=8, max_batch=reserved) as t:
            t.find_or_put(k[:1 << 19], out)
            t.rebuild(6 * n)
            check_dump_r3(b.u64(t.dump()), Oracle(keys[:1 << 19]).dump(), t.size())
            t.clear()
            before = free_bytes()
            assert "tile_insert" in routes(lambda: t.find_or_put(k, out))
            used = before - free_bytes()
            # unreserved, the first call's workspace (of half the keys) grows to this one's
            assert (used == 0) if reserved else used >= 5 * n
            assert out.all() and t.size() == n
