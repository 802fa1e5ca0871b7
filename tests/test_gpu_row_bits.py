"""A row's bits are its own: other queries of its wavefront, loud ones, infinite ones or none at all, leave no trace, whatever the keys make
its softmax reference do; and a row comes out the same in whatever chunk it is computed, where lserve_probe_prefill_shape names one
shape for both calls and neither has scratch."""
import numpy as np
import pytest
import torch

from helpers import block_mask_csr

pytestmark = pytest.mark.gpu

SINK, LOCAL = 128, 512


def _lib():
    import paper_2502_14866_amd as L

    L.load_library()
    return L


def _loudness(n):
    """Keys grow along a sequence, with a loud one now and then: sums of weights pass any bound again and again."""
    t = torch.arange(n)
    return torch.where(t % 150 == 149, 4.0 + 8.0 * t / n, 0.3 + 3.0 * t / n)[:, None, None]


def _inputs(L, heads, kv_heads, lengths, dtype, seed=5):
    dt = {"fp16": torch.float16, "bf16": torch.bfloat16}[dtype]
    desc = L.AttnDesc(heads, kv_heads, [1] * (kv_heads // 2) + [0] * (kv_heads - kv_heads // 2), dtype=dt, sink_tokens=SINK,
                      local_tokens=LOCAL)
    g = torch.Generator().manual_seed(seed)
    rnd = lambda n, h: torch.randn((n, h, 128), generator=g)
    k = torch.cat([rnd(n, kv_heads) * _loudness(n) for n in lengths]).to(dt).cuda()
    return desc, rnd(sum(lengths), heads).to(dt).cuda(), k, rnd(sum(lengths), kv_heads).to(dt).cuda()


def _i32(a):
    return torch.tensor(a, dtype=torch.int32, device="cuda")


def _cu(lengths):
    return _i32([0] + np.cumsum(lengths).tolist())


def _changed(q, how):
    """Half of the rows given other queries, and the rows that were left alone."""
    some = torch.rand(q.shape[0], generator=torch.Generator().manual_seed(11)) < 0.5
    other = q.clone()
    at = some.to(q.device)
    other[at] = q[at] * 16 if how == "loud" else float(how)
    return other, (~some).to(q.device)


def _same_rows(call, q, how):
    """call(q) -> (out, lse): equal in the rows that keep their queries, not a number in those that are none."""
    other, left = _changed(q, how)
    (a, la), (b, lb) = call(q), call(other)
    torch.cuda.synchronize()
    assert not torch.isnan(a).any() and not torch.isnan(la).any()
    assert torch.equal(a[left].view(torch.int16), b[left].view(torch.int16)) and torch.equal(la[:, left], lb[:, left])
    if how == "loud":
        assert not torch.isnan(b).any() and not torch.equal(a[~left], b[~left])
    else:
        assert torch.isnan(b[~left]).all()


def _buffers(q):
    return torch.full_like(q, float("nan")), torch.full((q.shape[1], q.shape[0]), float("nan"), device=q.device)


HOW = pytest.mark.parametrize("how", ["loud", "nan", "inf"])
TYPES = pytest.mark.parametrize("dtype", ["fp16", "bf16"])


@HOW
@TYPES
@pytest.mark.parametrize("heads,kv_heads,lengths,slices,half", [
    (64, 8, (1100, 77, 640), 1, 1),
    (32, 8, (4000,), 1, 1),          # the longest walk first
    (32, 8, (1500,), 2, 0),
    (8, 8, (4500, 1), 4, 0),
    (16, 8, (12001, 64), 1, 0),
    (8, 2, (51, 7, 33), 1, 0),
])
def test_prompts(heads, kv_heads, lengths, slices, half, dtype, how):
    L = _lib()
    desc, q, k, v = _inputs(L, heads, kv_heads, lengths, dtype)
    plan = L.lserve_probe_prefill_plan(desc, len(lengths), sum(lengths), max(lengths))
    assert (plan["dense"], plan["half"]) == (slices, half)

    def call(q):
        out, lse = _buffers(q)
        L.lserve_sparse_prefill(desc, q, k, v, _cu(lengths), max(lengths), out, lse)
        return out, lse
    _same_rows(call, q, how)


@HOW
@TYPES
@pytest.mark.parametrize("heads,kv_heads,lengths,thin,walk", [
    (32, 8, (5000, 500), False, 0), (24, 8, (2500, 70), True, 1), (32, 8, (2600,), True, 2)])
def test_listed_masks(heads, kv_heads, lengths, thin, walk, dtype, how):
    L = _lib()
    desc, q, k, v = _inputs(L, heads, kv_heads, lengths, dtype)
    masks = [lambda b, i: [j for j in range(i + 1) if j == i or ((7 * j + 3 * i) % (5 if thin else 9) == 0) == thin],
             lambda b, i: [j for j in range(i + 1) if j == i or ((j + i) % (3 if thin else 7) == 0) == thin]]
    qts, rp, cl, rows = block_mask_csr(masks, lengths)
    bm = L.BlockMask(_i32([-1] * 10 + [h % 2 for h in range(heads - 10)]), _i32(qts), _i32(rp), _i32(cl), 2, rows)
    assert L.lserve_probe_mask_walk(desc, len(lengths), sum(lengths), max(lengths), 2, rows, len(cl)) == walk
    ws = torch.empty((L.lserve_masked_prefill_workspace_bytes(desc, len(lengths), sum(lengths), max(lengths), 2, len(cl)),),
                     dtype=torch.uint8, device="cuda")

    def call(q):
        out, lse = _buffers(q)
        L.lserve_sparse_prefill_masked(desc, bm, q, k, v, _cu(lengths), max(lengths), out, lse, ws)
        return out, lse
    _same_rows(call, q, how)


def _cache(L, desc, k, v, hist, pages, bits):
    """One sequence's first `hist` tokens in pages of their own."""
    heads = desc.num_kv_heads
    if bits == 16:
        pool = lambda: torch.full((pages, heads, 64, 128), float("nan"), dtype=k.dtype, device="cuda")
    else:
        pool = lambda: torch.full((pages, heads, 64 * 128 * bits // 8 + 256), 0xff, dtype=torch.uint8, device="cuda")
    stats = torch.zeros((pages, heads, 4, 2, 128), dtype=k.dtype, device="cuda")
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(2)).to(torch.int32).reshape(1, -1).cuda()
    kv = L.PagedKV(pool(), pool(), stats, table, _i32([hist]), kv_bits=bits)
    L.lserve_append_kv(desc, kv, k[:hist].contiguous(), v[:hist].contiguous(), _i32([0, hist]), _i32([0]), hist)
    return kv


@HOW
@pytest.mark.parametrize("dtype,bits", [("fp16", 16), ("bf16", 16), ("bf16", 8), ("fp16", 4)])
@pytest.mark.parametrize("heads,kv_heads,hist,fresh,pieces,expand", [
    (32, 8, 14100, 190, 1, 0),       # in pieces, streaming heads beside the fold
    (32, 8, 16001, 512, 1, 1),       # over quantised pages turned into 16-bit ones
    (64, 8, 2047, 400, 0, 1),
    (32, 8, 101, 600, 0, 0),
])
def test_chunks(heads, kv_heads, hist, fresh, pieces, expand, dtype, bits, how):
    L = _lib()
    desc, q, k, v = _inputs(L, heads, kv_heads, (hist + fresh,), dtype)
    pages = -(-(hist + fresh) // 64)
    kv = _cache(L, desc, k, v, hist, pages, bits)
    q, kn, vn = q[hist:].contiguous(), k[hist:].contiguous(), v[hist:].contiguous()
    plan = L.lserve_probe_prefill_plan(desc, 1, fresh, fresh, pages, bits)
    assert bool(plan["pieces"]) == bool(pieces) and plan["expand"] == (expand and bits != 16)
    for scratch in (None, torch.empty((0,), dtype=torch.uint8, device="cuda")):
        def call(q):
            out, lse = _buffers(q)
            L.lserve_sparse_prefill_chunk(desc, kv, q, kn, vn, _i32([0, fresh]), fresh, out, lse, scratch=scratch)
            return out, lse
        _same_rows(call, q, how)


@TYPES
@pytest.mark.parametrize("heads,kv_heads,n,cuts,slices,half", [
    (64, 8, 2100, (13, 77, 203, 333, 509), 1, 1),
    (32, 8, 4200, (13, 77, 203, 333), 1, 1),      # the longest walk first
    (32, 8, 2100, (13, 77, 203), 2, 0),
    (8, 8, 1500, (13, 77, 203, 509), 4, 0),
    (32, 8, 9000, (77, 333, 2051), 1, 0),
])
def test_a_row_is_the_same_in_every_chunk(heads, kv_heads, n, cuts, slices, half, dtype):
    """The whole prompt in one call, and cut off the rows that wavefronts begin and end on: the rows in front as a shorter prompt, those
    behind as a chunk over the others."""
    L = _lib()
    desc, q, k, v = _inputs(L, heads, kv_heads, (n,), dtype)
    pages, none = -(-n // 64), torch.empty((0,), dtype=torch.uint8, device="cuda")
    shape = L.lserve_probe_prefill_shape(desc, 1, n, n)
    assert shape[0] == slices and L.lserve_probe_prefill_plan(desc, 1, n, n)["half"] == half
    out, lse = _buffers(q)
    L.lserve_sparse_prefill(desc, q, k, v, _i32([0, n]), n, out, lse)
    seen = 0
    for cut in cuts:
        assert L.lserve_probe_prefill_shape(desc, 1, n - cut, n - cut, pages) == shape
        kv = _cache(L, desc, k, v, cut, pages, 16)
        part, part_lse = _buffers(q[cut:])
        L.lserve_sparse_prefill_chunk(desc, kv, q[cut:].contiguous(), k[cut:].contiguous(), v[cut:].contiguous(), _i32([0, n - cut]),
                                      n - cut, part, part_lse, scratch=none)
        torch.cuda.synchronize()
        assert torch.equal(part.view(torch.int16), out[cut:].view(torch.int16)) and torch.equal(part_lse, lse[:, cut:]), cut
        m = n - cut
        if L.lserve_probe_prefill_shape(desc, 1, m, m) == shape:
            part, part_lse = _buffers(q[:m])
            L.lserve_sparse_prefill(desc, q[:m].contiguous(), k[:m].contiguous(), v[:m].contiguous(), _i32([0, m]), m, part, part_lse)
            torch.cuda.synchronize()
            assert torch.equal(part.view(torch.int16), out[:m].view(torch.int16)) and torch.equal(part_lse, lse[:, :m]), m
            seen += 1
    assert seen
