"""Performance cases: what a program does with these hash tables, each pass through the public entry points.

A pass that inserts starts by emptying its table, so that it can be repeated on the same state.  The keys of one
find-or-put call that are not in the table yet are pairwise distinct, except in the explorations: which copy of a
repeated absent key reports "new" is unspecified, and the flags would not be comparable.  Repeats of keys stored by
earlier calls are in every batched fill.  All outputs are membership flags and counts, exact whole numbers, so there is
no rounding to compare with a 64-bit result.

Families (the "op" of a case):
  call     one find-or-put of n keys into an empty table, then n queries, about half of them members
  fill     a long key sequence inserted in batches (10% repeats of earlier keys), then one batch of queries
  query    queries alone, against a table filled beforehand
  vectors  as fill, with state vectors of 2 or 4 words as keys
  explore  breadth-first exploration of a 16-process model, then a check which of some states were reached
  tables   many resident tables filled by one prepared many-table launch, then queried together
"""
from types import SimpleNamespace

import numpy as np
import torch

from paper_1712_09494_amd import binding as b
from paper_1712_09494_amd import inputs

DEV = "cuda"

# Levels of the exploration of the seed-1 model from its all-zero state: successors generated, states new.
LEVEL_SUCCESSORS = (48, 2156, 49501, 771837, 9166988, 88228274, 715127564)
LEVEL_NEW = (45, 1034, 16123, 191393, 1840442, 14900556, 104260775)


def listed():
    return [
        # the smallest calls: a small model's whole state set, default table; launches and latency count
        dict(name="small_bucketed", op="call", kind="bucketed", n=1000, capacity=2048, nhash=3, bucket_slots=16),
        dict(name="small_cuckoo", op="call", kind="cuckoo", n=4097, capacity=8192, nhash=3, bucket_slots=0),
        # ordinary ones: 2^20 keys at load factor 0.5 in a table that stays in the last-level cache, and a ragged count
        dict(name="set_bucketed", op="call", kind="bucketed", n=1 << 20, capacity=1 << 21, nhash=3, bucket_slots=16),
        dict(name="set_cuckoo", op="call", kind="cuckoo", n=1000003, capacity=1 << 21, nhash=3, bucket_slots=0),
        # the scaling workload: 2^26 keys in batches of 2^20 into a 0.7 GB table, both designs as the benchmark runs them
        dict(name="fill_bucketed", op="fill", kind="bucketed", n=1 << 26, batch=1 << 20, load=0.7, nhash=3,
             bucket_slots=8),
        dict(name="fill_cuckoo", op="fill", kind="cuckoo", n=1 << 26, batch=1 << 20, load=0.7, nhash=4,
             bucket_slots=0),
        # membership checks alone on such a table, half of them hits
        dict(name="query_bucketed", op="query", kind="bucketed", n=(1 << 24) + 77, members=60397978, load=0.7, hit=0.5,
             nhash=3, bucket_slots=8),
        # state vectors of 256 and 128 bits, in batches
        dict(name="vectors_bucketed", op="vectors", kind="bucketed", words=4, n=1 << 22, batch=1 << 20, load=0.7,
             nhash=3, bucket_slots=8),
        dict(name="vectors_cuckoo", op="vectors", kind="cuckoo", words=2, n=3000001, batch=1 << 20, load=0.7,
             nhash=3, bucket_slots=0),
        # explorations: the default split levels over all seven levels (813 M successors), and fused Cuckoo levels
        dict(name="explore_bucketed", op="explore", kind="bucketed", levels=7, fused=False, load=0.7, nhash=3,
             bucket_slots=8),
        dict(name="explore_fused_cuckoo", op="explore", kind="cuckoo", levels=6, fused=True, load=0.7, nhash=4,
             bucket_slots=0),
        # many resident tables of both designs, 2^10 to 2^22 slots, filled by one launch and queried together
        dict(name="tables_mixed", op="tables", tables=64, log_min=10, log_max=22, load=0.6, nhash=3, bucket_slots=8),
    ]


def draw(rng):
    op = rng.choice(("call", "call", "call", "fill", "fill", "query", "vectors", "explore", "tables"))
    kind = rng.choice(("bucketed", "cuckoo"))
    load = rng.choice((0.5, 0.6, 0.7, 0.8, 0.9))
    nhash = rng.choice((3, 4)) if kind == "bucketed" or load < 0.85 else 4
    case = dict(op=op, kind=kind, nhash=nhash, bucket_slots=rng.choice((8, 16, 16, 32)) if kind == "bucketed" else 0)
    if op == "call":
        n = int(2 ** rng.uniform(8, 24)) | rng.randint(0, 1)
        return dict(case, n=n, capacity=int(n / load) + 1)
    if op == "fill":
        n = int(2 ** rng.uniform(18, 25.5)) | rng.randint(0, 1)
        return dict(case, n=n, batch=int(2 ** rng.uniform(14, 24)) | rng.randint(0, 1), load=load)
    if op == "query":
        return dict(case, n=int(2 ** rng.uniform(8, 24)) | rng.randint(0, 1), members=int(2 ** rng.uniform(12, 25.5)),
                    load=load, hit=rng.choice((0.0, 0.5, 1.0)))
    if op == "vectors":
        n = int(2 ** rng.uniform(12, 22)) | rng.randint(0, 1)
        return dict(case, words=rng.choice((2, 4)), n=n, batch=int(2 ** rng.uniform(12, 21)) | rng.randint(0, 1),
                    load=min(load, 0.8))
    if op == "explore":
        return dict(case, levels=rng.choice((4, 5, 6)), fused=rng.choice((False, True)), load=min(load, 0.8))
    hi = rng.randint(14, 22)
    return dict(op="tables", tables=rng.randint(8, 64), log_min=rng.randint(8, 12), log_max=hi, load=min(load, 0.8),
                nhash=rng.choice((3, 4)), bucket_slots=rng.choice((8, 16, 32)))


# ---- inputs, made on the GPU from the seed --------------------------------------------------------------------

def _shr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _signed(c):
    return c - (1 << 64) if c >> 63 else c


def _mix(x):
    """A bijection on 64-bit words (the MurmurHash3 finalizer), so distinct indices give distinct keys."""
    x = (x ^ _shr(x, 33)) * _signed(0xFF51AFD7ED558CCD)
    x = (x ^ _shr(x, 33)) * _signed(0xC4CEB9FE1A85EC53)
    return x ^ _shr(x, 33)


def _keys(idx, seed, word=0):
    return _mix(idx ^ (((seed % (1 << 20)) + 1) << 40) ^ (word << 36))


def _rows(idx, seed, words):
    """State vectors: the first word names the vector, the others are shared by 16, 256, ... neighbours, as the
    components of successive states are."""
    if words == 1:
        return _keys(idx, seed)
    return torch.stack([_keys(idx >> (4 * j), seed, j + 1) for j in range(words)], dim=1).contiguous()


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _sequence(n, batch, repeats, seed):
    """Indices of a key sequence: fresh indices in increasing order, and from the second batch on a share of repeats
    drawn from the fresh indices of earlier batches.  Returns (indices, number of distinct)."""
    g = _gen(seed)
    pos = torch.arange(n, device=DEV)
    rep = (torch.rand(n, device=DEV, generator=g) < repeats) & (pos >= batch)
    count = torch.cumsum(~rep, 0)
    before = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), count])[pos // batch * batch]
    old = (torch.rand(n, device=DEV, generator=g, dtype=torch.float64) * before).long()
    return torch.where(rep, old, count - 1), int(count[-1])


def _probe(n, members, hit, seed):
    """Query indices: a share of members, the rest never inserted."""
    g = _gen(seed + 1)
    is_hit = torch.rand(n, device=DEV, generator=g) < hit
    some = (torch.rand(n, device=DEV, generator=g, dtype=torch.float64) * members).long()
    return torch.where(is_hit, some, members + torch.arange(n, device=DEV))


def _table(case, capacity, seed, batch, **kw):
    if case["kind"] == "bucketed":
        kw["bucket_slots"] = case["bucket_slots"]
    return b.Table(case["kind"], capacity=capacity, nhash=case["nhash"], seed=seed, max_batch=batch, **kw)


def _flags(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def _distinct(case):
    """About how many distinct keys a fill of this case holds."""
    return case["n"] if case["n"] <= case["batch"] else int(case["n"] - 0.1 * (case["n"] - case["batch"]))


def _relabelled(seed):
    """The seed-1 model with its processes reordered and their local states renamed: another input, the same number of
    states and successors at every level."""
    base = inputs.BfsModel(1)
    rng = np.random.default_rng(seed)
    place = rng.permutation(16)
    name = [rng.permutation(16) for _ in range(16)]
    local = [None] * 16
    for p in range(16):
        rows = [None] * 16
        for s in range(16):
            rows[name[p][s]] = [int(name[p][t]) for t in base.local[p][s]]
        local[place[p]] = rows
    syncs = []
    for (p, q, pe, qe) in base.syncs:
        pr, qr = [None] * 16, [None] * 16
        for s in range(16):
            pr[name[p][s]] = [int(name[p][t]) for t in pe[s]]
            qr[name[q][s]] = [int(name[q][t]) for t in qe[s]]
        syncs.append((int(place[p]), int(place[q]), pr, qr))
    initial = 0
    for p in range(16):
        initial |= int(name[p][0]) << (4 * int(place[p]))
    return SimpleNamespace(local=local, syncs=syncs), initial


def _walks(model, initial, n, levels, seed):
    """n states at the ends of random walks of 1 .. 2 * levels local transitions from the initial state."""
    rng = np.random.default_rng(seed + 1)
    count = np.array([[len(t) for t in row] for row in model.local])
    target = np.zeros((16, 16, 4), dtype=np.uint64)
    for p in range(16):
        for s in range(16):
            target[p, s, :count[p, s]] = model.local[p][s]
    st = np.full(n, initial, dtype=np.uint64)
    steps = rng.integers(1, 2 * levels + 1, n)
    for k in range(2 * levels):
        p = rng.integers(0, 16, n)
        sh = (4 * p).astype(np.uint64)
        s = ((st >> sh) & np.uint64(15)).astype(np.int64)
        t = target[p, s, rng.integers(0, 1 << 30, n) % count[p, s]]
        st = np.where(k < steps, (st & ~(np.uint64(15) << sh)) | (t << sh), st)
    return torch.from_numpy(st.view(np.int64)).to(DEV)


def _table_sizes(case):
    """Capacities spread evenly over the logarithm of the range, odd ones among them."""
    m = case["tables"]
    lo, hi = case["log_min"], case["log_max"]
    return [int(2 ** (lo + (hi - lo) * (i + 0.5) / m)) for i in range(m)]


def prepare(case, seed):
    op = case["op"]
    if op == "call":
        n = case["n"]
        t = _table(case, case["capacity"], seed, n)
        return SimpleNamespace(op=op, table=t, keys=_keys(torch.arange(n, device=DEV), seed),
                               probe=_keys(_probe(n, n, 0.5, seed), seed))
    if op in ("fill", "vectors"):
        n, batch, words = case["n"], min(case["batch"], case["n"]), case.get("words", 1)
        idx, distinct = _sequence(n, batch, 0.1, seed)
        t = _table(case, int(distinct / case["load"]) + 1, seed, batch, key_words=words)
        return SimpleNamespace(op=op, table=t, n=n, batch=batch, keys=_rows(idx, seed, words), out=_flags(n),
                               probe=_rows(_probe(batch, distinct, 0.5, seed), seed, words))
    if op == "query":
        m = case["members"]
        t = _table(case, int(m / case["load"]) + 1, seed, min(m, 1 << 24))
        for lo in range(0, m, 1 << 24):
            t.find_or_put(_keys(torch.arange(lo, min(m, lo + (1 << 24)), device=DEV), seed))
        return SimpleNamespace(op=op, table=t, probe=_keys(_probe(case["n"], m, case["hit"], seed), seed),
                               out=_flags(case["n"]))
    if op == "explore":
        model, initial = _relabelled(seed)
        states = 1 + sum(LEVEL_NEW[:case["levels"]])
        t = _table(case, int(states / case["load"]) + 1, seed, 0)
        return SimpleNamespace(op=op, table=t, model=model, initial=initial, levels=case["levels"], fused=case["fused"],
                               probe=_walks(model, initial, 1 << 16, case["levels"], seed))
    # tables: even ones bucketed, odd ones Cuckoo, each filled to the load factor by its own batch
    tables, keys, probes = [], [], []
    for i, cap in enumerate(_table_sizes(case)):
        n = max(1, int(cap * case["load"]))
        kind = dict(kind="bucketed", bucket_slots=case["bucket_slots"]) if i % 2 == 0 else dict(kind="cuckoo")
        tables.append(_table(dict(kind, nhash=case["nhash"]), cap, seed + i, n))
        keys.append(_keys(torch.arange(n, device=DEV) + (i << 24), seed))
        probes.append(_keys(_probe(n, n, 0.5, seed + i) + (i << 24), seed))
    total = sum(k.numel() for k in keys)
    ends = np.cumsum([k.numel() for k in keys])
    new, found = _flags(total), _flags(total)
    outs = [new[e - k.numel():e] for e, k in zip(ends, keys)]
    answers = [found[e - k.numel():e] for e, k in zip(ends, keys)]
    return SimpleNamespace(op=op, tables=tables, probes=probes, answers=answers, new=new, found=found,
                           plan=b.MultiPlan(tables, keys, outs))


# ---- one pass ---------------------------------------------------------------------------------------------------

def run(state):
    s = state
    if s.op == "call":
        s.table.clear()
        return {"new": s.table.find_or_put(s.keys), "found": s.table.query(s.probe)}
    if s.op in ("fill", "vectors"):
        s.table.clear()
        for lo in range(0, s.n, s.batch):
            hi = min(lo + s.batch, s.n)
            s.table.find_or_put(s.keys[lo:hi], s.out[lo:hi])
        return {"new": s.out, "found": s.table.query(s.probe)}
    if s.op == "query":
        return {"found": s.table.query(s.probe, s.out)}
    if s.op == "explore":
        s.table.clear()
        r = s.table.bfs_explore(s.model, s.levels, s.initial, fused=s.fused)
        return {"successors": np.array(r["batch_sizes"]), "new": np.array(r["new_counts"]),
                "reached": s.table.query(s.probe)}
    for t in s.tables:
        t.clear()
    s.plan.launch()
    b.query_multi(s.tables, s.probes, s.answers)
    return {"new": s.new, "found": s.found}


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def work(case):
    """Bytes: keys read and flags written once, the emptied table written once, every stored key written once (and a
    queried table's looked-up words read once); the hashing is a few integer operations per key."""
    op = case["op"]
    if op == "call":
        n = case["n"]
        return {"bytes": 2 * n * 9 + 8 * case["capacity"] + 8 * n + 8 * n, "flops": 0}
    if op in ("fill", "vectors"):
        w, q, d = case.get("words", 1), min(case["batch"], case["n"]), _distinct(case)
        return {"bytes": (case["n"] + q) * (8 * w + 1) + 8 * d / case["load"] + 8 * w * d + 8 * q, "flops": 0}
    if op == "query":
        return {"bytes": case["n"] * (8 + 1 + 8), "flops": 0}
    if op == "explore":
        new = sum(LEVEL_NEW[:case["levels"]])
        # each state is written once to the table and once as frontier, and read once from there
        return {"bytes": 8 * new / case["load"] + 3 * 8 * new + (1 << 16) * 17, "flops": 0}
    caps = _table_sizes(case)
    n = sum(int(c * case["load"]) for c in caps)
    return {"bytes": 8 * sum(caps) + 8 * n + n * (9 + 9 + 8), "flops": 0}
