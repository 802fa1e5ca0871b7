"""How calls on chunks use scratch: what it may change and what it must not."""
import random

import pytest

import paper_2502_14866_amd as L
import paper_2502_14866_amd.binding as B
from paper_2502_14866_amd.binding import LserveError


def _sizes(seed, n):
    rng = random.Random(seed)
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    for _ in range(n):
        heads, kv_heads = rng.choice([(32, 8), (32, 32), (8, 2), (64, 8), (32, 16), (12, 4), (24, 8)])
        flags = rng.choice([[1] * (kv_heads // 2) + [0] * (kv_heads - kv_heads // 2), [0] * kv_heads])
        batch, longest, width = log(1, 12), log(1, 4096), log(2, 4096)
        total = rng.choice([batch * longest, longest + rng.randint(0, (batch - 1) * longest)])
        yield L.AttnDesc(heads, kv_heads, flags), batch, total, longest, width + longest // 64 + 1, rng.choice([16, 8, 4])


def test_no_rows_sums_are_taken_in_fewer_key_ranges_with_scratch_than_without():
    """Weights are rounded to 16 bits relative to the maximum of their range: fewer ranges, larger errors (against 64 bits 2.78e-3
    for a streaming head in four slices, 2.84e-3 in one)."""
    used = {"pieces": 0, "expand": 0, "apart": 0}
    for args in _sizes(5, 4000):
        bare, plan = B.lserve_probe_prefill_plan(*args, scratch=False), B.lserve_probe_prefill_plan(*args)
        assert bare["pieces"] == bare["expand"] == 0
        assert plan["dense"] >= bare["dense"], (args, bare, plan)
        assert plan["streaming"] >= bare["streaming"] or not any(args[0].streaming_flags), (args, bare, plan)
        assert (B.lserve_chunk_scratch_bytes(*args) > 0) == bool(plan["pieces"] or plan["expand"])
        for k in used:
            used[k] += bool(plan[k])
    assert all(n >= 100 for n in used.values()), used  # the sizes reach all of it


@pytest.mark.parametrize("args", [
    (8, 2, 4, 3912, 978, 36, 4),     # slices folded for both classes over quantised pages, for dense heads only over expanded ones
    (32, 16, 1, 2583, 2583, 207, 8),  # one slice over quantised pages, two over expanded ones
    (64, 8, 1, 962, 962, 707, 8),
])
def test_expanded_pages_keep_the_slices_of_both_classes(args):
    heads, kv_heads, *sizes = args
    desc = L.AttnDesc(heads, kv_heads, [1 if h < kv_heads // 2 else 0 for h in range(kv_heads)])
    bare, plan = B.lserve_probe_prefill_plan(desc, *sizes, scratch=False), B.lserve_probe_prefill_plan(desc, *sizes)
    assert plan["dense"] >= bare["dense"] and plan["streaming"] >= bare["streaming"]


def test_prompts_have_neither():
    plan = B.lserve_probe_prefill_plan(L.AttnDesc(32, 8, [1] * 4 + [0] * 4), 1, 4096, 4096)
    assert plan == {"dense": 1, "streaming": 1, "half": 1, "pieces": 0, "apart": 0, "expand": 0}


def test_arguments():
    desc = L.AttnDesc(8, 2, [1, 0])
    for bad in ((0, 1, 1, 0, 16), (1, 0, 1, 0, 16), (1, 10, 11, 0, 16), (1, 10, 10, -1, 16), (1, 10, 10, 4, 5)):
        with pytest.raises(LserveError):
            B.lserve_probe_prefill_plan(desc, *bad)
    with pytest.raises(LserveError):
        B.lserve_probe_prefill_plan(L.AttnDesc(8, 2, [1, 0], page_size=32), 1, 10, 10)


# (heads, KV heads, sequences of one length): by half workgroups or by whole ones.  Beside each case its time, us, by half workgroups and by whole
# ones; where the other one is the quicker the rule, which is older than these times, has not been fitted again.
@pytest.mark.parametrize("heads,kv_heads,batch,length,half", [
    (32, 8, 1, 4096, 1),     # 111 and 117
    (32, 32, 10, 327, 1),    # 31.8 and 40.6
    (32, 16, 1, 51, 0),      # 6.8 and 6.9: one tile
    (32, 8, 4, 64, 0),       # 7.2 and 7.5
    (32, 32, 1, 51, 1),      # 6.8 and 7.0
    (64, 8, 16, 128, 0),     # 24.3 and 25.6: two full rounds of walks of two tiles
    (64, 8, 16, 70, 1),      # 17.7 and 19.4
    (64, 8, 13, 215, 1),     # 35.6 and 42.0
    (32, 8, 4, 399, 0),      # 18.0 and 19.4: one full round of some tiles each
    (32, 8, 8, 231, 0),      # 15.6 and 16.2
    (32, 8, 16, 123, 1),     # 12.7 and 13.8
    (32, 8, 2, 1024, 1),     # 30.8 and 34.1
    (32, 32, 4, 385, 0),     # 18.9 and 19.5
    (32, 32, 6, 385, 1),     # 25.9 and 30.6
    (32, 32, 18, 3001, 0),   # 1263 and 1150: 27 rounds, no groups
    (32, 32, 21, 1888, 1),   # 691 and 632
    (32, 32, 5, 3017, 1),    # 300 and 304
    (32, 8, 1, 65536, 0),    # 16.1 ms and 15.5 ms
])
def test_half_workgroups_where_they_are_quicker(heads, kv_heads, batch, length, half):
    desc = L.AttnDesc(heads, kv_heads, [1] * (kv_heads // 2) + [0] * (kv_heads // 2))
    assert B.lserve_probe_prefill_plan(desc, batch, batch * length, length)["half"] == half


@pytest.mark.parametrize("heads,kv_heads,batch,length,half", [  # no streaming head
    (32, 32, 18, 3001, 0),   # 2269 and 1601: more dense heads than XCDs, in many rounds
    (32, 32, 64, 500, 0),    # 388 and 308
    (32, 16, 18, 3001, 0),   # 1601 and 1426
    (32, 16, 16, 2000, 1),   # 659 and 628
    (32, 32, 4, 2000, 1),    # 150 and 153
    (32, 8, 16, 2000, 1),    # 574 and 582
    (32, 8, 2, 2000, 0),     # 74.8 and 74.0: two rounds of long walks
    (32, 8, 1, 2500, 1),     # 66.6 and 69.5
])
def test_half_workgroups_without_streaming_heads(heads, kv_heads, batch, length, half):
    desc = L.AttnDesc(heads, kv_heads, [0] * kv_heads)
    assert B.lserve_probe_prefill_plan(desc, batch, batch * length, length)["half"] == half


def test_half_workgroups_of_streaming_heads_alone():
    desc = L.AttnDesc(32, 8, [1] * 8)
    assert B.lserve_probe_prefill_plan(desc, 8, 16000, 2000)["half"] == 1  # 166 and 178
    assert B.lserve_probe_prefill_plan(desc, 1, 51, 51)["half"] == 0       # 7.0 and 7.3


@pytest.mark.parametrize("heads,kv_heads,lengths,first", [
    (32, 8, (4096,), 1),        # 104 us with priority, 109 without
    (32, 8, (3500,), 1),        # 88.6 and 92.5
    (32, 32, (3500,), 1),       # 84.4 and 88.1
    (32, 8, (4600,), 1),        # 122.5 and 125.8: two and a quarter workgroups to a unit
    (32, 8, (4609,), 0),
    (32, 32, (4900,), 0),       # 136.8 and 134.8
    (32, 8, (4000, 500), 1),    # 100.7 and 105.5
    (32, 8, (3500, 1500), 0),   # 98.5 and 95.4
    (32, 8, (2000, 2000), 0),   # 62.8 and 63.1: walks of 32 tiles
    (16, 8, (3000,) * 3, 0),    # 90.0 and 88.4: of 47
    (64, 8, (4096,), 0),        # 189.9 and 185.5
    (32, 8, (3000,), 0),        # goes in key slices
])
def test_priority_where_the_longest_walk_decides(heads, kv_heads, lengths, first):
    desc = L.AttnDesc(heads, kv_heads, [1] * (kv_heads // 2) + [0] * (kv_heads // 2))
    assert B.lserve_probe_prefill_longest_first(desc, len(lengths), sum(lengths), max(lengths)) == first


def test_priority_arguments():
    desc = L.AttnDesc(8, 2, [1, 0])
    for bad in ((0, 1, 1), (1, 0, 1), (1, 10, 11), (1, 10, 0)):
        with pytest.raises(LserveError):
            B.lserve_probe_prefill_longest_first(desc, *bad)
    with pytest.raises(LserveError):
        B.lserve_probe_prefill_longest_first(L.AttnDesc(8, 2, [1, 0], page_size=32), 1, 10, 10)
