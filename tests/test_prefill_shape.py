"""The shape the host chooses for a prefill launch: key slices, which heads fold them, what a workgroup's units are."""
import pytest

import paper_2502_14866_amd as L
from paper_2502_14866_amd.binding import LserveError


def _shape(heads, kv_heads, batch, total, longest, pages=0, bits=16, **kw):
    desc = L.AttnDesc(heads, kv_heads, [1 if h < kv_heads // 2 else 0 for h in range(kv_heads)], **kw)
    return L.lserve_probe_prefill_shape(desc, batch, total, longest, pages, bits)


# (heads, KV heads, sequences, rows, longest, pages, bits): key slices of the quickest shape, measured in all of them
@pytest.mark.parametrize("sizes,slices", [
    ((32, 8, 1, 65536, 65536, 0, 16), 1),    # 15.4 ms in one slice, 17.6 in two
    ((8, 2, 1, 2272, 2272, 0, 16), 4),       # 30 us in four, 65 in one
    ((32, 8, 5, 200, 123, 0, 16), 1),        # walks of two tiles: nothing to share out
    ((32, 8, 1, 512, 512, 520, 16), 4),      # 363 us in four, 849 in one
    ((32, 8, 1, 2635, 2635, 751, 16), 1),    # one round of workgroups: 1229 us; in four slices two rounds: 1513
    ((32, 8, 1, 2043, 2043, 649, 16), 1),    # likewise 1060 and 1284
    ((32, 32, 4, 2356, 589, 1034, 16), 1),   # likewise 1844 and 2791
    ((32, 8, 2, 1970, 1357, 231, 8), 1),     # likewise 510, in two 619
    ((32, 8, 1, 512, 512, 520, 8), 2),       # 714 us in two, 1108 in one
])
def test_slices_of_launches_with_a_clear_winner(sizes, slices):
    assert _shape(*sizes)[0] == slices


@pytest.mark.parametrize("heads,kv_heads", [(32, 8), (8, 8), (64, 8), (12, 4), (5, 1)])
def test_every_shape_is_one_the_kernels_are_built_for(heads, kv_heads):
    for batch, longest in ((1, 1), (1, 64), (1, 777), (1, 40000), (3, 65), (16, 4096), (64, 300), (65, 128), (200, 1)):
        for total in {batch * longest, longest + batch - 1}:
            for pages in (0, 1, 64, 4096, 65536):
                for bits in (16, 8, 4):
                    slices, fold_dense, fold_stream, one_head = _shape(heads, kv_heads, batch, total, longest, pages, bits)
                    assert slices in ((1, 2, 4) if bits == 16 or pages == 0 else (1, 2))
                    assert fold_dense == (slices > 1) and fold_stream <= fold_dense and one_head in (0, 1)


def test_layers_of_one_kind_of_head():
    for flags in ([0] * 8, [1] * 8):
        desc = L.AttnDesc(32, 8, flags)
        assert L.lserve_probe_prefill_shape(desc, 1, 65536, 65536)[0] == 1
        assert L.lserve_probe_prefill_shape(desc, 2, 300, 200, 700, 4)[0] in (1, 2)


def test_arguments():
    for bad in ((0, 1, 1, 0, 16), (1, 0, 1, 0, 16), (1, 10, 11, 0, 16), (1, 10, 10, -1, 16), (1, 10, 10, 4, 5)):
        with pytest.raises(LserveError):
            _shape(8, 2, *bad)
    with pytest.raises(LserveError):
        _shape(8, 2, 1, 10, 10, page_size=32)
