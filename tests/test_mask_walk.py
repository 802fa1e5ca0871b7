"""Which way a prefill under a listed mask goes: merged lists, the caller's rows in four key slices, or in half workgroups."""
import pytest

import paper_2502_14866_amd as L
from paper_2502_14866_amd.binding import LserveError

MERGED, SLICES, HALVES = 0, 1, 2


def walk(heads, kv_heads, lengths, density, masks=2, **kw):
    """Of masks whose rows keep a first tile, a band of four and `density` of the rest."""
    desc = L.AttnDesc(heads, kv_heads, [1 if h < kv_heads // 2 else 0 for h in range(kv_heads)], **kw)
    tiles = [-(-n // 64) for n in lengths]
    kept = sum(min(i, 3) + 1 + max(0, i - 3) * density for t in tiles for i in range(t))
    return L.lserve_probe_mask_walk(desc, len(lengths), sum(lengths), max(lengths), masks, sum(tiles), int(masks * kept))


@pytest.mark.parametrize("heads,kv_heads,lengths,density", [
    (32, 8, (1342,), 0.42), (8, 2, (7393,), 0.25), (8, 2, (5101,), 0.35), (32, 16, (1100,), 0.2), (32, 8, (900,), 0.3)])
def test_slices_stay_slices_where_half_workgroups_are_quicker_still(heads, kv_heads, lengths, density):
    """One slice instead of four makes the error against 64 bits about 1 % larger."""
    assert walk(heads, kv_heads, lengths, density) == SLICES


@pytest.mark.parametrize("heads,kv_heads,lengths,density", [
    (32, 8, (12345,), 0.3), (64, 8, (6330, 6330), 0.08), (32, 8, (2907, 2907), 0.3), (32, 8, (519, 519), 0.4)])
def test_merged_lists_give_way_to_half_workgroups(heads, kv_heads, lengths, density):
    assert walk(heads, kv_heads, lengths, density) == HALVES


def test_lists_that_keep_most_tiles_are_merged():
    assert walk(32, 8, (12345,), 0.8) == MERGED
    assert walk(24, 8, (9000,), 0.95, masks=3) == MERGED


def test_arguments():
    desc = L.AttnDesc(8, 2, [1, 0])
    good = [1, 100, 100, 1, 2, 3]
    assert L.lserve_probe_mask_walk(desc, *good) in (MERGED, SLICES, HALVES)
    for at, bad in ((0, 0), (1, 0), (2, 0), (2, 101), (3, 0), (4, 0), (5, -1)):
        args = list(good)
        args[at] = bad
        with pytest.raises(LserveError):
            L.lserve_probe_mask_walk(desc, *args)
    with pytest.raises(LserveError):
        L.lserve_probe_mask_walk(L.AttnDesc(8, 2, [1, 0], page_size=32), *good)
