"""GPU: Cuckoo batches into small tables (one block, the table in LDS), at the
edges of the rule, against the oracle: flags per call, stored set, queries,
every key at one of its slots with the earlier ones taken.  The kernel timing
says which kernels ran."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_dump_r3, check_flags_r2, check_query_r1  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.array(a).view(np.int64)).cuda()


def run(t, o, keys, expect):
    b.ht_timing_enable(True)
    out = t.find_or_put(dev(keys))
    names = set(b.ht_timing_report())
    b.ht_timing_enable(False)
    assert expect in names, names
    check_flags_r2(keys, out.cpu().numpy(), o.find_or_put(keys), f"n={keys.size}")


# n, distinct, slots, hash functions, flags, kernel of the first call and of the same keys again
CASES = [
    (1, 1, 16, 3, 0, "cuckoo_whole", "cuckoo_whole"),
    (65, 60, 128, 4, 0, "cuckoo_whole", "cuckoo_whole"),
    (1024, 900, 8192, 2, 0, "cuckoo_whole", "cuckoo_whole"),
    (1025, 900, 8192, 2, 0, "cuckoo_probe", "cuckoo_probe"),
    (1000, 900, 1300, 3, b.HT_FLAG_CUCKOO_LOOKAHEAD, "cuckoo_whole", "cuckoo_whole"),
    (1024, 500, 1024, 8, 0, "cuckoo_whole", "cuckoo_whole"),
    (4096, 4096, 8192, 3, b.HT_FLAG_CHAIN_STATS, "cuckoo_whole", "cuckoo_whole"),
    (4097, 4000, 4800, 4, 0, "cuckoo_whole", "cuckoo_probe"),         # load factor 0.83
    (8192, 7000, 8192, 4, 0, "cuckoo_whole", "cuckoo_probe"),
    (8193, 7000, 8192, 4, 0, "cuckoo_probe", "cuckoo_probe"),
    (4000, 3000, 8208, 3, 0, "cuckoo_probe", "cuckoo_probe"),         # one slot row too many
]


@pytest.mark.parametrize("n,distinct,cap,nhash,flags,first,again", CASES)
def test_small_cuckoo_tables(n, distinct, cap, nhash, flags, first, again):
    keys = inputs.random_sequence(n, distinct, seed=n + cap)
    if n > 100:
        keys[3::97] = np.uint64(b.EMPTY)
    more = inputs.random_sequence(max(1, n // 8), max(1, n // 10), seed=n + cap + 1)
    o = Oracle()
    with b.Table("cuckoo", capacity=cap, nhash=nhash, flags=flags, stash_slots=4096) as t:
        run(t, o, keys, first)
        run(t, o, keys[::-1], again)
        run(t, o, more, "cuckoo_whole" if t.stats()["capacity"] <= 8192 and more.size <= 1024 else "cuckoo_probe")
        check_dump_r3(b.u64(t.dump()), o.dump(), t.size())
        probe = np.concatenate([keys, more, inputs.uniform_keys(2000, seed=n)])
        check_query_r1(t.query(dev(probe)).cpu().numpy(), o.query(probe))
        st = t.stats()
        assert st["lost"] == 0
        raw = b.u64(t.dump_raw())
        slots, stash = raw[:st["capacity"]], set(raw[st["capacity"]:].tolist())
        taken = slots != np.uint64(b.EMPTY)
        at = {int(k): i for i, k in enumerate(slots) if taken[i]}
        for k in o.dump()[:1500].tolist():
            if k == b.EMPTY or k in stash:
                continue
            h = [t.hash_index(k, j) for j in range(nhash)]
            assert at[k] in h
            if len(set(h)) == nhash:
                assert taken[h[:h.index(at[k])]].all()
        if flags & b.HT_FLAG_CHAIN_STATS:
            hist = b.ht_chain_histogram(t.handle)
            # every exchange but a chain's last one evicts a key
            assert sum(i * c for i, c in enumerate(hist["counts"])) - hist["chains"] == st["evictions"]


def test_small_cuckoo_overflow_keeps_every_key():
    """Far more keys than slots: chains end in the stash, then on the overflow
    list; every key stays a member."""
    keys = inputs.uniform_keys(1000, seed=5)
    with b.Table("cuckoo", capacity=256, nhash=3, stash_slots=64) as t:
        flags = t.find_or_put(dev(keys)).cpu().numpy()
        assert (flags == 1).all()
        assert t.query(dev(keys)).all() and t.sync_status() == b.HT_EFULL
        assert t.size() == 1000
