"""GPU: tables whose blocks allocate all the LDS that a block can have run every
kernel of their find-or-put, also those that work in LDS themselves (Cuckoo
state vectors reach the evict kernel here), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle, VecOracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def table(kind, lds, **kw):
    """A table with the most LDS per block that is accepted, less `lds`."""
    for most in (160 << 10, 64 << 10):
        try:
            return b.Table(kind, lds_bytes=most - lds, **kw)
        except b.HtError as e:
            err = e
    raise err


CASES = [("bucketed", dict(bucket_slots=8)), ("bucketed", dict(bucket_slots=64)),
         ("bucketed", dict(bucket_slots=16, flags=b.HT_FLAG_BUCKETED_ONE_LANE)), ("cuckoo", dict()),
         ("bucketed", dict(bucket_slots=8, key_words=2)), ("cuckoo", dict(key_words=2)), ("cuckoo", dict(key_words=4))]


@pytest.mark.parametrize("lds", [0, 16, 4096])
@pytest.mark.parametrize("kind,kw", CASES)
def test_all_of_a_blocks_lds(kind, kw, lds):
    w, n = kw.get("key_words", 1), 5000
    o = Oracle() if w == 1 else VecOracle(w)
    keys = inputs.uniform_keys(n, seed=7) if w == 1 else inputs.vector_of_index(np.arange(n), w, seed=7)
    k = torch.from_numpy(np.ascontiguousarray(keys).view(np.int64)).cuda()
    with table(kind, lds, capacity=int(n / 0.85), nhash=4, stash_slots=4096, **kw) as t:
        for lo in range(0, n, 2500):
            part = slice(lo, lo + 2500)
            assert (t.find_or_put(k[part]).cpu().numpy() == o.find_or_put(keys[part])).all()
        assert not t.find_or_put(k).any() and t.query(k).all() and t.size() == n
