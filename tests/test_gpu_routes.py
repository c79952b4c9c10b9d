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


def block_each():
    """Lanes of one block of 256 threads on each compute unit."""
    return torch.cuda.get_device_properties(0).multi_processor_count * 256


@pytest.mark.parametrize("width", [8, 16, 32, 64])
def test_lanes_need_keys_and_room(width):
    """Second batches (the tiled passes take first ones): groups below half a
    block of keys per compute unit, and where the table lacks the slots for
    each key in flight (six blocks per compute unit at most)."""
    one, full = block_each(), 6 * block_each()
    cases = [(one // 2 - 1, 64 * one, "groups"), (one // 2, 64 * one, "lanes"), (4096, 1 << 20, "groups")]
    room = min(width, 32)
    for n, slots in ((one, room * one), (4 * one, room * 4 * one), (full - 1, room * full)):
        cases += [(n, slots, "lanes"), (n, slots - room * width, "groups")]
    room = 16 if width in (8, 64) else 32
    for n in (full, 2 * full):
        cases += [(n, room * full, "lanes"), (n, room * full - width, "groups")]
    for n, slots, form in cases:
        with b.Table("bucketed", capacity=slots, nhash=3, bucket_slots=width) as t:
            assert t.stats()["capacity"] == slots
            keys, o = inputs.uniform_keys(n, seed=n), Oracle()
            served(t, o, keys)
            r = served(t, o, keys)
            assert r == {"bucketed_fop": 1, f"bucketed_fop.{form}": 1}, (n, slots, r)


@pytest.mark.parametrize("width", [8, 16, 32, 64])
def test_lanes_need_a_table_with_free_slots(width):
    """Groups once more than a share of the slots was put, larger for more
    keys; lanes again once the table was handed as many keys as it has slots,
    for calls that fill the grid of six blocks."""
    one = block_each()
    for n, eighths in ((one // 2, 5 if width == 8 else 2), (one, 5 if width == 8 else 4), (6 * one, 5), (16 * one, 7)):
        with b.Table("bucketed", capacity=32 * n, nhash=3, bucket_slots=width) as t:
            slots = t.stats()["capacity"]
            keys = dev(inputs.uniform_keys(n, seed=3))
            for puts in range(0, 36 * n, n):
                r = routes(lambda: t.find_or_put(keys))
                lanes = puts <= slots // 8 * eighths or (puts >= slots and n >= 6 * one)
                assert r == {"bucketed_fop": 1, f"bucketed_fop.{'lanes' if lanes else 'groups'}": 1}, (n, puts, r)
            f = t.find_or_put(keys)
            assert not f.any() and t.size() == n
