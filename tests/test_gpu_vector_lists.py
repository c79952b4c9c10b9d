"""GPU: state-vector find-or-put at the edges of its eight-slot claim steps and
of the evict kernel's gathered lists (none, a few, one and several turns of 64
leftovers in a wave), against the oracle: flags, stored rows, queries."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import VecOracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from test_gpu_vector import check_dump, check_flags, fop, query  # noqa: E402

pytestmark = pytest.mark.gpu

# kind, words, bucket slots, members, members stored by the first call, keys of the second call, load, hash functions
CASES = [
    ("cuckoo", 2, 0, 1 << 20, 7 << 17, (1 << 20) + 77, 0.9, 4),    # 129 keys a wave, over half of the new ones left over
    ("cuckoo", 4, 0, 700001, 600000, 524289, 0.9, 4),              # 65 keys a wave
    ("cuckoo", 2, 0, 3000, 1, 64, 0.3, 3),                         # nothing left over
    ("cuckoo", 4, 0, 5000, 2500, 4999, 0.95, 4),
    ("bucketed", 2, 8, 40000, 30000, 33333, 0.98, 3),
    ("bucketed", 4, 16, 40000, 20000, 40000, 0.97, 2),
    ("bucketed", 2, 32, 70001, 35000, 50001, 0.98, 1),
    ("bucketed", 4, 64, 70001, 65000, 65537, 0.99, 3),
]


@pytest.mark.parametrize("kind,w,width,members,first,n,load,nhash", CASES)
def test_claims_and_leftovers(kind, w, width, members, first, n, load, nhash):
    rng = np.random.default_rng(members + n)
    pool = inputs.vector_of_index(np.arange(members), w, seed=w, structured=bool(nhash % 2))
    kw = dict(bucket_slots=width) if width else {}
    o = VecOracle(w)
    with b.Table(kind, capacity=int(members / load), nhash=nhash, key_words=w, stash_slots=65536, **kw) as t:
        for part in (pool[:first], pool[np.sort(rng.integers(0, members, size=n))], pool[rng.permutation(members)]):
            check_flags(part, fop(t, part), o.find_or_put(part), w, f"{kind} {part.shape[0]}")
        q = np.concatenate([pool[:5000], inputs.vector_of_index(np.arange(10 ** 7, 10 ** 7 + 2000), w, seed=w)])
        assert (query(t, q) == o.query(q)).all()
        check_dump(t, o, w, kind)
