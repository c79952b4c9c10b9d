"""GPU: which kernels serve a find-or-put, from the timing report: the names
tell the forms of one kernel apart, and the rules that choose between forms
are looked at on both sides of their edges.  Flags against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import Oracle  # noqa: E402
from paper_1712_09494_amd import binding as b  # noqa: E402
from paper_1712_09494_amd import inputs  # noqa: E402
from parity import check_flags_r2  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def routes(call):
    """The names that a call adds to the timing report, with their launches."""
    b.ht_timing_enable(True)
    call()
    r = {k: v[0] for k, v in b.ht_timing_report().items()}
    b.ht_timing_enable(False)
    return r


def served(t, o, keys):
    out = {}
    r = routes(lambda: out.update(f=t.find_or_put(dev(keys))))
    check_flags_r2(keys, out["f"].cpu().numpy(), o.find_or_put(keys), f"n={keys.size}")
    return r


def test_names_tell_lanes_from_groups():
    keys = inputs.uniform_keys(3000, seed=1)
    for kw, names in ((dict(keys_per_group=1), {"bucketed_fop", "bucketed_fop.groups"}),
                      (dict(flags=b.HT_FLAG_BUCKETED_ATOMIC_LOADS), {"bucketed_fop", "bucketed_fop.groups"}),
                      (dict(flags=b.HT_FLAG_BUCKETED_ONE_LANE), {"bucketed_lane_fop"})):
        with b.Table("bucketed", capacity=40000, nhash=3, bucket_slots=16, **kw) as t:
            assert served(t, Oracle(), keys) == dict.fromkeys(names, 1)
    # the form's time is in the name before the dot, once
    with b.Table("bucketed", capacity=40000, nhash=3, bucket_slots=16) as t:
        b.ht_timing_enable(True)
        t.find_or_put(dev(keys))
        r = b.ht_timing_report()
        b.ht_timing_enable(False)
        assert r["bucketed_fop"][1] > 0 and r["bucketed_fop.groups"] == (1, 0.0)
    n = 1 << 20                                # lanes, whichever rule chooses them
    with b.Table("bucketed", capacity=40 * n, nhash=3, bucket_slots=16) as t:
        r = served(t, Oracle(), inputs.uniform_keys(n, seed=2))
        assert r == {"bucketed_fop": 1, "bucketed_fop.lanes": 1}


@pytest.mark.parametrize("width", [8, 64])
@pytest.mark.parametrize("per_group", [0, 1, 2, 4])
def test_keys_per_group_asks_for_the_groups(width, per_group):
    """First batches that an ordinary table takes in LDS, by a single call and
    by a plan."""
    for n, cap, whole in ((1000, 4096, "tile_whole"), (1 << 18, 1 << 19, "tile_insert")):
        keys = inputs.uniform_keys(n, seed=n)
        with b.Table("bucketed", capacity=cap, nhash=3, bucket_slots=width, keys_per_group=per_group) as t:
            r = served(t, Oracle(), keys)
            assert r == {"bucketed_fop": 1, "bucketed_fop.groups": 1} if per_group else whole in r
            t.clear()
            out = torch.empty(n, dtype=torch.uint8, device="cuda")
            plan = b.MultiPlan([t], [dev(keys)], [out])
            assert routes(plan.launch) == {"multi_fill" if per_group else "multi_tiles": 1}
            assert out.all() and t.size() == n
            plan.close()


@pytest.mark.parametrize("width", [8, 16, 64])
def test_lanes_need_many_keys_and_room(width):
    """Groups below a key for each lane of four blocks per compute unit, where
    the table has less than 16 slots a key, and where three quarters of its
    slots (seven eighths for a full grid) would not hold what was put; lanes again once it was handed as many
    keys as it has slots, for calls that fill the grid of six blocks."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    lanes, full = cus * 4 * 256, cus * 6 * 256
    for n, cap, form in ((lanes - 1, 16 * lanes, "groups"), (lanes, 16 * lanes, "lanes"),
                         (lanes, 16 * lanes - width, "groups"), (4096, 1 << 20, "groups"), (40000, 1 << 20, "groups")):
        with b.Table("bucketed", capacity=cap, nhash=3, bucket_slots=width) as t:
            r = served(t, Oracle(), inputs.uniform_keys(n, seed=n))
            assert r == {"bucketed_fop": 1, f"bucketed_fop.{form}": 1}, (n, cap)
    for n in (full, full - 1):
        keys = inputs.uniform_keys(n, seed=1)
        with b.Table("bucketed", capacity=3 * n, nhash=3, bucket_slots=width) as t:
            o = Oracle()
            slots, puts = t.stats()["capacity"], 0
            for k in range(5):
                r = served(t, o, keys)
                form = "lanes" if puts >= slots and n == full else "groups"
                assert set(r) == ({"bucketed_fop", f"bucketed_fop.{form}"} if k else
                                  {"tile_partition", "tile_insert", "tile_finish"}), (k, r)
                puts += n
    for n, eighths in ((lanes, 6), (full, 7)):
        with b.Table("bucketed", capacity=16 * n, nhash=3, bucket_slots=width) as t:
            most = t.stats()["capacity"] // 8 * eighths
            keys = dev(inputs.uniform_keys(n, seed=3))
            for puts in range(0, 16 * n, n):
                r = routes(lambda: t.find_or_put(keys))
                assert ("bucketed_fop.lanes" in r) == (puts <= most) and "bucketed_fop" in r, (puts, r)


@pytest.mark.parametrize("width", [8, 16, 64])
def test_lanes_from_a_block_per_unit_in_a_roomy_table(width):
    """Lanes also from one block per compute unit on, where the table has 64
    slots a key and half of its slots would hold what was put."""
    n = torch.cuda.get_device_properties(0).multi_processor_count * 256
    for m, cap, form in ((n, 64 * n, "lanes"), (n - 1, 64 * n, "groups"), (n, 64 * n - width, "groups")):
        with b.Table("bucketed", capacity=cap, nhash=3, bucket_slots=width) as t:
            keys = inputs.uniform_keys(m, seed=5)
            assert t.stats()["capacity"] == cap
            o, most = Oracle(), cap // 2
            for puts in range(0, 40 * m, m):
                if puts % (4 * m) and puts + m < most:
                    t.find_or_put(dev(keys))
                    continue
                r = served(t, o, keys)
                want = form if puts <= most else "groups"
                assert r == {"bucketed_fop": 1, f"bucketed_fop.{want}": 1}, (m, cap, puts)
