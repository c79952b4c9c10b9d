"""GPU: a large first batch that repeats a few of its keys, which the partition
leaves out of the tiles: flags, stored set and queries against the oracle at
chunk and tile edges, by single calls and plans, and the time beside a batch
of different keys (2^22 copies of one key took 25 times as long when one block
served them all)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_flags_r2  # noqa: E402
from test_gpu_hot_keys import dev, hot, kernel_us  # noqa: E402
from test_gpu_tile import check_table, run  # noqa: E402

pytestmark = pytest.mark.gpu

# keys, what repeats, slots per key, bucket width, hash functions, odd flag address
CASES = [
    (1 << 18, "one", 2.0, 8, 3, 0), ((1 << 18) + 1, "few", 1.4, 16, 3, 1), ((1 << 20) + 4095, "half", 2.0, 64, 2, 3),
    ((1 << 21) - 1, "blocks", 7.9, 8, 3, 0), ((1 << 21) + 1, "one", 1.2, 32, 3, 0), ((1 << 21) + 8191, "few", 2.0, 8, 1, 2),
    (1 << 22, "half", 7.99, 8, 3, 0), (3 << 20, "blocks", 1.5, 16, 4, 0),
]


@pytest.mark.parametrize("n,how,room,width,nhash,off", CASES)
def test_copies_in_a_first_batch(n, how, room, width, nhash, off):
    keys = inputs.key_of_index(hot(n, how, n), seed=width)
    keys[7::5003] = np.uint64(b.EMPTY)
    o = Oracle()
    with b.Table("bucketed", capacity=int(n * room), nhash=nhash, bucket_slots=width) as t:
        first = np.concatenate([keys[:500], inputs.uniform_keys(100, seed=1)])
        run(t, o, first, "bucketed_fop")
        run(t, o, keys, "tile_insert", off)                    # some keys already stored
        check_table(t, o, width, np.concatenate([keys[:4000], inputs.uniform_keys(4000, seed=n + 1)]))


def test_runs_just_within_and_beyond_a_chunks_share():
    """Copies of one key in every chunk around the number at which the
    partition begins to leave them out."""
    n, chunk, tiles = 1 << 18, 4096, 256
    share = 2 * (chunk // tiles) + 16
    for m in (share - 17, share, share + 1, chunk):
        i = np.arange(n)
        keys = inputs.key_of_index(np.where(i % chunk < m, n, i), seed=m)
        o = Oracle()
        with b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=8) as t:
            run(t, o, keys, "tile_insert")
            check_table(t, o, 8, keys[:6000])


def test_copies_of_keys_that_overflow():
    """A table whose buckets and stash cannot hold the batch: a copy of a key
    that was kept on the overflow list answers as it does or as a later copy."""
    n = 1 << 18
    keys = inputs.key_of_index(hot(n, "half", 3), seed=9)
    kw = dict(nhash=1, bucket_slots=8, stash_slots=64, bucket_walk=1, overflow_slots=1 << 17)
    with b.Table("bucketed", capacity=int(1.4 * n), flags=b.HT_FLAG_BUCKETED_PAPER_FULL, **kw) as t:
        f = t.find_or_put(dev(keys)).cpu().numpy()
        d = np.unique(keys)
        new, over = keys[f == 1], np.unique(keys[f == 2])
        assert np.unique(new).size == new.size and new.size + over.size == d.size and over.size
        assert not np.intersect1d(new, over).size and t.query(dev(keys)).all() and t.size() == d.size


def test_plan_with_copies():
    rng = np.random.default_rng(4)
    tables, keys = [], []
    for k, (n, width) in enumerate([(5000, 8), (9000, 16), (70001, 8), (70001, 64), (300000, 8)]):
        tables.append(b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=width))
        keys.append(inputs.key_of_index(hot(n, ("one", "few", "half", "blocks", "half")[k], k), seed=k)[rng.permutation(n)])
    outs = [torch.full((k.size,), 9, dtype=torch.uint8, device="cuda") for k in keys]
    plan = b.MultiPlan(tables, [dev(k) for k in keys], outs)
    for _ in range(2):
        b.ht_timing_enable(True)
        plan.launch()
        assert "multi_tiles" in b.ht_timing_report()
        b.ht_timing_enable(False)
        for t, k, out in zip(tables, keys, outs):
            o = Oracle()
            check_flags_r2(k, out.cpu().numpy(), o.find_or_put(k), f"n={k.size}")
            check_table(t, o, t.stats()["bucket_slots"], k[:2000])
            t.clear()
    plan.close()
    for t in tables:
        t.close()


@pytest.mark.parametrize("n", [1 << 18, 1 << 22])
@pytest.mark.parametrize("how", ["one", "few", "half"])
def test_copies_take_no_longer(n, how):
    with b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=8, max_batch=n) as t:
        different = kernel_us(t, dev(inputs.key_of_index(np.arange(n), seed=4)))
        copies = kernel_us(t, dev(inputs.key_of_index(hot(n, how, 4), seed=4)))
    print(f"{n} {how}: different keys {different:.1f} us, copies {copies:.1f} us")
    assert copies < 3 * different
