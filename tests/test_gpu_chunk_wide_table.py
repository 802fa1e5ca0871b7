"""Chunks behind page tables far wider than their sequences: pieces are chosen for the histories that a table has room for, and where the
sequences turn out short their dense walks stay whole, with the bits of the call without scratch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _call(L, heads, kv_heads, hist, fresh, wide, bits, dtype, written=False):
    """-> plan, outputs with scratch, outputs without."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(23)
    rnd = lambda *s: torch.randn(s, generator=g, device=dev).to(dtype)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    cu = lambda xs: i32([0] + torch.tensor(xs).cumsum(0).tolist())
    B, own = len(hist), max(-(-(h + n) // 64) for h, n in zip(hist, fresh))
    desc = L.AttnDesc(heads, kv_heads, [1] * (kv_heads // 2) + [0] * (kv_heads - kv_heads // 2), dtype=dtype)
    if bits == 16:
        pool = lambda: torch.full((B * own, kv_heads, 64, 128), float("nan"), dtype=dtype, device=dev)
    else:
        pool = lambda: torch.full((B * own, kv_heads, 64 * 128 * bits // 8 + 256), 0xff, dtype=torch.uint8, device=dev)
    table = torch.full((B, own * wide), 2 ** 30, dtype=torch.int32, device=dev)  # past the sequences: no pages at all
    table[:, :own] = torch.randperm(B * own, generator=g, device=dev).to(torch.int32).reshape(B, own)
    stats = torch.zeros((B * own, kv_heads, 4, 2, 128), dtype=dtype, device=dev)
    kv = L.PagedKV(pool(), pool(), stats, table, i32(hist), kv_bits=bits)
    L.lserve_append_kv(desc, kv, rnd(sum(hist), kv_heads, 128), rnd(sum(hist), kv_heads, 128), cu(hist), i32([0] * B), max(hist))
    q, k, v = rnd(sum(fresh), heads, 128), rnd(sum(fresh), kv_heads, 128), rnd(sum(fresh), kv_heads, 128)
    got = []
    for scratch in (None, torch.empty((0,), dtype=torch.uint8, device=dev)):
        out, lse = torch.full_like(q, float("nan")), torch.full((heads, q.shape[0]), float("nan"), device=dev)
        if written:  # the chunk is in the pages as well
            L.lserve_append_kv(desc, kv, k, v, cu(fresh), i32(hist), max(fresh))
            kv.seq_lens = i32([h + n for h, n in zip(hist, fresh)])
            L.lserve_sparse_prefill_paged(desc, kv, q, cu(fresh), max(fresh), own * wide * 64, out, lse, scratch=scratch)
        else:
            L.lserve_sparse_prefill_chunk(desc, kv, q, k, v, cu(fresh), max(fresh), out, lse, scratch=scratch)
        got.append((out, lse))
    torch.cuda.synchronize()
    assert not any(torch.isnan(x).any() for pair in got for x in pair)
    return L.lserve_probe_prefill_plan(desc, B, sum(fresh), max(fresh), own * wide, bits), got


@pytest.mark.parametrize("dtype,bits,written", [(torch.float16, 16, True), (torch.bfloat16, 16, False), (torch.float16, 8, False),
                                                (torch.bfloat16, 4, False)])
@pytest.mark.parametrize("heads,kv_heads,hist,fresh,wide", [
    (64, 8, (1214,) * 7, (17, 2, 5, 11, 3, 8, 6), 32),
    (32, 8, (589, 1, 64, 300), (3, 3, 70, 1), 32),   # an end inside the first page, on one
    (8, 8, (530,), (274,), 32),                      # no groups: a block is four tiles
    (12, 2, (700, 128), (33, 0), 32),                # six heads per group; an idle sequence
    (32, 16, (503, 503, 503), (113, 66, 39), 32),
])
def test_short_sequences_stay_whole(heads, kv_heads, hist, fresh, wide, dtype, bits, written):
    import paper_2502_14866_amd as L

    L.load_library()
    plan, ((a, la), (b, lb)) = _call(L, heads, kv_heads, hist, fresh, wide, bits, dtype, written)
    assert plan["pieces"] and plan["apart"] and not plan["expand"]
    assert torch.equal(a, b) and torch.equal(la, lb)


@pytest.mark.parametrize("bits", [16, 8])
def test_from_one_to_the_other(bits):
    """Histories from a page to what the table has room for: whole up to some length, in pieces from there on."""
    import paper_2502_14866_amd as L

    L.load_library()
    whole = []
    for pages in (1, 3, 9, 17, 31, 47, 64, 96, 128, 192, 256):
        plan, ((a, la), (b, lb)) = _call(L, 32, 8, (pages * 64 - 5,), (40,), 257 // pages, bits, torch.float16)
        assert plan["pieces"] and plan["apart"]
        whole.append(torch.equal(a, b) and torch.equal(la, lb))
        # weights and outputs are rounded to fp16 on both sides: 2^-11 of the largest output twice; sums of rounded weights: 2^-11
        assert (a.float() - b.float()).abs().max() <= 2 ** -10 * a.float().abs().max() and (la - lb).abs().max() <= 2 ** -11
    assert whole[0] and not whole[-1] and whole == sorted(whole, reverse=True)
