"""GPU: the find-or-put of a large first batch (partition, tile and finish
passes) and of a batch into a small table (one block, the table in LDS), at
the edges of their chunks, tiles and rules, against the oracle: flags per
call, stored set, queries, and slots that fill each bucket as a prefix.  The
kernel timing says which kernels ran."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_dump_r3, check_flags_r2, check_query_r1  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def batch_of(n, distinct, seed, empty=False):
    k = inputs.random_sequence(n, distinct, seed=seed)
    if empty:
        k[7::5003] = np.uint64(b.EMPTY)          # the all-ones key, many times
    return k


def run(t, o, keys, expect_kernel, out_offset=0):
    buf = torch.full((keys.size + out_offset,), 9, dtype=torch.uint8, device="cuda")
    b.ht_timing_enable(True)
    out = t.find_or_put(dev(keys), buf[out_offset:])
    names = set(b.ht_timing_report())
    b.ht_timing_enable(False)
    assert expect_kernel in names, names
    check_flags_r2(keys, out.cpu().numpy(), o.find_or_put(keys), f"n={keys.size}")


def check_table(t, o, bucket_slots, probe):
    check_dump_r3(b.u64(t.dump()), o.dump(), t.size())
    check_query_r1(t.query(dev(probe)).cpu().numpy(), o.query(probe))
    st = t.stats()
    raw = b.u64(t.dump_raw())[:st["capacity"]].reshape(-1, bucket_slots)
    full = raw != np.uint64(b.EMPTY)
    assert (full[:, :-1] >= full[:, 1:]).all(), "a bucket is not filled as a prefix"
    assert st["lost"] == 0 and st["overflow_count"] == 0


# n, share of distinct keys, slots per key, bucket width, hash functions, flags, all-ones keys, odd flag address
TILED = [
    (1 << 18, 1.0, 1.4, 8, 3, 0, False, 0),                    # the smallest batch, nearly the fullest table
    ((1 << 18) + 1, 0.9, 2.0, 16, 3, 0, True, 1),              # one key in the last chunk, unaligned flags
    ((1 << 18) + 4095, 0.5, 7.9, 8, 1, 0, False, 3),           # one hash function, nearly the emptiest table
    ((1 << 20) - 1, 0.8, 1.45, 64, 2, 0, True, 0),
    (1 << 20, 1.0, 1.13, 32, 4, 0, False, 0),                  # load factor 0.88: many full buckets
    ((1 << 20) + 4097, 0.95, 2.3, 8, 3, b.HT_FLAG_BUCKETED_PAPER_FULL, False, 2),
    ((1 << 21) - 1, 0.9, 3.0, 16, 3, 0, False, 0),             # the last batch with chunks of 4096
    ((1 << 21) + 8191, 0.9, 1.5, 8, 3, 0, True, 1),            # chunks of 8192
    (1 << 22, 0.7, 7.99, 8, 3, 0, False, 0),                   # nearly the most tiles
]


@pytest.mark.parametrize("n,share,room,width,nhash,flags,empty,off", TILED)
def test_tiled_first_batch(n, share, room, width, nhash, flags, empty, off):
    keys = batch_of(n, int(n * share), n ^ width, empty)
    cap = int(n * room)
    o = Oracle()
    if flags & b.HT_FLAG_BUCKETED_PAPER_FULL:
        # keys of full buckets go straight to the stash: room for all of them
        kw = dict(stash_slots=65536)
    else:
        kw = {}
    with b.Table("bucketed", capacity=cap, nhash=nhash, bucket_slots=width, flags=flags, **kw) as t:
        first = keys[:1000]
        run(t, o, first, "bucketed_fop" if t.stats()["capacity"] > 8192 else "tile_whole")
        run(t, o, keys, "tile_insert", off)                    # some keys already stored
        run(t, o, keys[::-1], "bucketed_fop")                  # not larger than what came before: direct
        probe = np.concatenate([keys[:4000], inputs.uniform_keys(4000, seed=n + 1)])
        check_table(t, o, width, probe)
        # empty again: the rule starts over, and no flags are asked for
        t.clear()
        b._check(b.load().ht_find_or_put(t.handle, dev(keys).data_ptr(), n, None,
                                         torch.cuda.current_stream().cuda_stream), "ht_find_or_put")
        torch.cuda.synchronize()
        check_dump_r3(b.u64(t.dump()), Oracle(keys).dump(), t.size())


@pytest.mark.parametrize("n,distinct,cap,width,nhash", [
    (512, 512, 8192, 8, 3), (513, 400, 512, 16, 3), (1023, 1000, 2048, 16, 1), (1025, 700, 1000, 64, 2),
    (2048, 2048, 8192, 32, 4), (2048, 500, 512, 8, 3), (2047, 2047, 2100, 8, 3),
])
def test_whole_small_table(n, distinct, cap, width, nhash):
    keys = batch_of(n, distinct, n + cap, True)
    o = Oracle()
    with b.Table("bucketed", capacity=cap, nhash=nhash, bucket_slots=width) as t:
        run(t, o, keys[:100], "bucketed_fop")
        run(t, o, keys, "tile_whole", 1)
        run(t, o, keys, "bucketed_fop")
        check_table(t, o, width, np.concatenate([keys, inputs.uniform_keys(1000, seed=n)]))


def test_whole_small_table_overflows():
    """More keys than slots and stash: every key is a member all the same,
    and the table says that it is full."""
    keys = inputs.uniform_keys(2000, seed=3)
    with b.Table("bucketed", capacity=512, nhash=2, bucket_slots=8, stash_slots=64) as t:
        flags = t.find_or_put(dev(keys)).cpu().numpy()
        assert (flags == 1).sum() == 512 + 64 and (flags == 2).sum() == 2000 - 576
        assert t.query(dev(keys)).all() and t.sync_status() == b.HT_EFULL
        check_dump_r3(b.u64(t.dump()), keys, t.size())


def test_captured_calls_stay_direct():
    """A call under capture uses no workspace of its own, so its replays do
    not depend on what later calls allocate."""
    n = 1 << 18
    keys = inputs.uniform_keys(n, seed=8)
    k, out = dev(keys), torch.empty(n, dtype=torch.uint8, device="cuda")
    with b.Table("bucketed", capacity=2 * n, nhash=3, bucket_slots=8) as t:
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            t.clear()
            t.find_or_put(k, out)
        for rep in range(3):
            out.fill_(7)
            g.replay()
            torch.cuda.synchronize()
            assert out.all() and t.size() == n, rep
            t.clear()
            assert t.find_or_put(k).all()                      # eager: the tiled passes
            big = dev(inputs.uniform_keys(n + 50000 * (rep + 1), seed=9))
            t.clear()
            t.find_or_put(big)                                 # a larger workspace
            assert t.size() == big.numel()


# capacity, keys, distinct, kind and options of a many-table plan: small tables (one block each), tables of several
# tiles, and ones the passes do not take (too empty, too full, flags, other kinds, no keys)
PLAN = [
    (700, 600, 500, "bucketed", dict(bucket_slots=8)), (8192, 7000, 7000, "bucketed", dict(bucket_slots=16)),
    (8200, 64, 64, "bucketed", dict(bucket_slots=8)), (8200, 5000, 4000, "bucketed", dict(bucket_slots=8)),
    (50001, 30001, 30000, "bucketed", dict(bucket_slots=32)), (300000, 180000, 150000, "bucketed", dict(bucket_slots=8)),
    (40000, 4097, 4097, "bucketed", dict(bucket_slots=64)), (1 << 20, 900, 900, "bucketed", dict(bucket_slots=8)),
    (1000, 3000, 400, "bucketed", dict(bucket_slots=16)), (20000, 9000, 8000, "cuckoo", {}),
    (30000, 15000, 15000, "bucketed", dict(bucket_slots=8, flags=b.HT_FLAG_BUCKETED_ONE_LANE)),
    (5000, 0, 0, "bucketed", dict(bucket_slots=8)), (6000, 3000, 2500, "bucketed", dict(bucket_slots=8, key_words=2)),
]


def plan_tables():
    tables, keys = [], []
    for i, (cap, n, d, kind, kw) in enumerate(PLAN):
        w = kw.get("key_words", 1)
        tables.append(b.Table(kind, capacity=cap, nhash=3, **kw))
        if w > 1:
            k = inputs.vector_sequence(n, d, w, seed=60 + i)
        else:
            k = inputs.random_sequence(n, d, seed=60 + i) if n else np.zeros(0, dtype=np.uint64)
            if n > 1000:
                k[11::977] = np.uint64(b.EMPTY)
        keys.append(np.ascontiguousarray(k))
    return tables, keys


def check_plan(tables, keys, outs, new):
    for t, k, o, (cap, n, d, kind, kw) in zip(tables, keys, outs, PLAN):
        f = o.cpu().numpy()[:n]
        if kw.get("key_words", 1) > 1:
            assert int(f.sum()) == (d if new else 0) and t.size() == d
            continue
        exp = Oracle() if new else Oracle(k)
        check_flags_r2(k, f, exp.find_or_put(k), f"cap={cap} n={n}")
        check_dump_r3(b.u64(t.dump()), exp.dump(), t.size(), f"cap={cap} n={n}")


def test_plan_with_tiled_tables():
    tables, keys = plan_tables()
    outs = [torch.full((max(n, 1),), 9, dtype=torch.uint8, device="cuda") for _, n, _, _, _ in PLAN]
    plan = b.MultiPlan(tables, [dev(k) for k in keys], outs)

    def launch(expect):
        b.ht_timing_enable(True)
        plan.launch()
        names = set(b.ht_timing_report())
        b.ht_timing_enable(False)
        assert (expect in names) and not ({"multi_tiles", "multi_fill"} - {expect}) & names, names

    launch("multi_tiles")                  # empty tables
    check_plan(tables, keys, outs, True)
    launch("multi_fill")                   # as much in them as the launch brings
    check_plan(tables, keys, outs, False)
    # cleared and launched in a graph, with eager work between the replays
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        for t in tables:
            t.clear()
        plan.launch(stream=s)
    for _ in range(3):
        for o in outs:
            o.fill_(9)
        g.replay()
        torch.cuda.synchronize()
        check_plan(tables, keys, outs, True)
        assert tables[5].query(dev(keys[5])).all()
        plan.launch()
        torch.cuda.synchronize()
        check_plan(tables, keys, outs, False)
    plan.close()
    for t in tables:
        t.close()
