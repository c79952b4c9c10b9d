"""GPU: batches in which a few keys come again and again: flags, stored set and
queries against the oracle, and the time beside a batch of different keys.
Compare-and-swaps of one slot are served one after another, so that a kernel
in which every copy of an absent key issues one takes tens of times as long
(2^18 copies of one key: 70 times)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle, VecOracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_dump_r3, check_flags_r2  # noqa: E402
from test_gpu_vector import check_dump, check_flags, fop, query  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def hot(n, how, seed):
    """Indices of n keys: one key, a few, half of them one key, or every
    second wave's worth of one key among different ones."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    if how == "one":
        return np.zeros(n, dtype=np.int64)
    if how == "few":
        return rng.integers(0, 100, size=n)
    if how == "half":
        return np.where(rng.random(n) < 0.5, n, i)
    return np.where(i // 64 % 2 == 0, i // 128 % 3, i + 3)


HOW = ("one", "few", "half", "blocks")


@pytest.mark.parametrize("how", HOW)
@pytest.mark.parametrize("kind,kw", [
    ("bucketed", dict(bucket_slots=8, flags=b.HT_FLAG_BUCKETED_ONE_LANE)),
    ("bucketed", dict(bucket_slots=64, nhash=1, flags=b.HT_FLAG_BUCKETED_ONE_LANE)),
    ("bucketed", dict(bucket_slots=16)), ("cuckoo", {})])
def test_copies_within_a_call(kind, kw, how):
    """Single calls and a plan, also where buckets are full and keys end in the
    stash."""
    n = 70001
    keys = inputs.key_of_index(hot(n, how, 5), seed=11)
    keys[5::4001] = np.uint64(b.EMPTY)
    kw = dict(dict(nhash=3, stash_slots=65536), **kw)
    for room in (1.02, 20.0):
        cap = int(np.unique(keys).size * room) + 64
        o = Oracle()
        with b.Table(kind, capacity=cap, **kw) as t, b.Table(kind, capacity=cap, **kw) as p:
            for part in (keys[:n // 3], keys):
                check_flags_r2(part, t.find_or_put(dev(part)).cpu().numpy(), o.find_or_put(part), f"{how} {room}")
            check_dump_r3(b.u64(t.dump()), o.dump(), t.size())
            out = torch.empty(n, dtype=torch.uint8, device="cuda")
            plan = b.MultiPlan([p], [dev(keys)], [out])
            plan.launch()
            check_flags_r2(keys, out.cpu().numpy(), Oracle().find_or_put(keys), f"plan {how} {room}")
            check_dump_r3(b.u64(p.dump()), o.dump(), p.size())
            plan.close()


@pytest.mark.parametrize("how", HOW)
@pytest.mark.parametrize("kind,w,width", [("bucketed", 2, 8), ("bucketed", 4, 64), ("cuckoo", 2, 0), ("cuckoo", 4, 0)])
def test_copies_of_vectors(kind, w, width, how):
    n = 30001
    v = inputs.vector_of_index(hot(n, how, 6), w, seed=3, structured=True)
    kw = dict(bucket_slots=width) if width else {}
    o = VecOracle(w)
    distinct = np.unique(v, axis=0).shape[0]
    with b.Table(kind, capacity=int(distinct * 1.1) + 64, nhash=4, key_words=w, stash_slots=65536, **kw) as t:
        for part in (v[:n // 3], v, v):
            check_flags(part, fop(t, part), o.find_or_put(part), w, how)
        assert (query(t, v) == 1).all()
        check_dump(t, o, w, how)


def test_overflowing_copies():
    """Copies of keys that fit neither their bucket nor the stash: the
    overflow list keeps them, and every one is a member."""
    keys = inputs.key_of_index(np.arange(4000) % 500, seed=2)
    with b.Table("bucketed", capacity=128, nhash=1, bucket_slots=8, stash_slots=64, bucket_walk=1,
                 flags=b.HT_FLAG_BUCKETED_ONE_LANE) as t:
        f = t.find_or_put(dev(keys)).cpu().numpy()
        assert set(np.unique(f)) == {0, 1, 2} and t.query(dev(keys)).all() and t.size() == 500
        new = np.unique(keys[f == 1])
        assert new.size == (f == 1).sum() and not set(new) & set(keys[f == 2])
        check_dump_r3(b.u64(t.dump()), np.unique(keys), t.size())


def kernel_us(t, keys):
    """Median kernel time of the find-or-put of `keys` into the emptied table."""
    out = []
    for _ in range(7):
        t.clear()
        b.ht_timing_enable(True)
        t.find_or_put(keys)
        out.append(sum(ms for _, ms in b.ht_timing_report().values()) * 1e3)
        b.ht_timing_enable(False)
    return float(np.median(out))


@pytest.mark.parametrize("kind,w,kw", [
    ("bucketed", 1, dict(bucket_slots=8, flags=b.HT_FLAG_BUCKETED_ONE_LANE)),
    ("bucketed", 1, dict(bucket_slots=64, flags=b.HT_FLAG_BUCKETED_ONE_LANE)),
    ("bucketed", 2, dict(bucket_slots=8)), ("bucketed", 4, dict(bucket_slots=16)), ("cuckoo", 4, {})])
def test_one_key_takes_no_longer(kind, w, kw):
    n = 1 << 18
    make = (lambda i: inputs.key_of_index(i, seed=4)) if w == 1 else (lambda i: inputs.vector_of_index(i, w, seed=4))
    with b.Table(kind, capacity=2 * n, nhash=3, key_words=w, max_batch=n, **kw) as t:
        different = kernel_us(t, dev(make(np.arange(n))))
        one = kernel_us(t, dev(make(np.zeros(n, dtype=np.int64))))
    print(f"{kind} {w} {kw}: different keys {different:.1f} us, one key {one:.1f} us")
    assert one < 4 * different
