"""Paths of their own for small calls: the write-back of one token per sequence, lists cut into many pieces, selection of
short sequences, and the quantiser's reciprocal."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload, make_decode_inputs

from parity import assert_attention_close

pytestmark = pytest.mark.gpu


def _lib():
    import paper_2502_14866_amd as L

    L.load_library()
    return L


@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("page,logical,kv_bits", [(64, 16, 16), (16, 16, 16), (32, 4, 16), (128, 16, 16), (64, 16, 8), (64, 8, 4)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_one_token_append_equals_the_general_write_back(dtype, page, logical, kv_bits, two_way):
    """The same call with max_new_per_seq 1 and 2 takes the one-token and the general kernel: the same bytes everywhere,
    at the first and last slot of pages and logical pages, with idle sequences among the others."""
    L = _lib()
    dev = torch.device("cuda:0")
    hkv, flags, local = 3, [0, 1, 0], 2 * page
    pos = [0, 1, logical - 1, logical, page - 1, page, 3 * page + 5, 4 * page - 1, 17]
    fresh = [1, 1, 1, 1, 1, 1, 1, 1, 0]
    B_, max_pages, ring = len(pos), 5, 1 + 2
    g = torch.Generator().manual_seed(3)
    table = torch.randperm(B_ * max_pages, generator=g).to(torch.int32).reshape(B_, max_pages).to(dev)
    ring_table = torch.randperm(B_ * ring, generator=g).to(torch.int32).reshape(B_, ring).to(dev)
    desc = L.AttnDesc(2 * hkv, hkv, flags, page_size=page, logical_page_size=logical, dtype=dtype, sink_tokens=page,
                      local_tokens=local)
    k = torch.randn((sum(fresh), hkv, 128), generator=g).to(dtype).to(dev)
    v = torch.randn((sum(fresh), hkv, 128), generator=g).to(dtype).to(dev)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(fresh)]), dtype=torch.int32, device=dev)
    start = torch.tensor(pos, dtype=torch.int32, device=dev)

    def pool(n, heads, seed):
        gg = torch.Generator().manual_seed(seed)
        if kv_bits == 16:
            return torch.randn((n, heads, page, 128), generator=gg).to(dtype).to(dev)
        return torch.randint(0, 256, (n, heads, 64 * 128 * kv_bits // 8 + 256), generator=gg, dtype=torch.uint8).to(dev)

    results = []
    for bound in (1, 2):
        heads = 2 if two_way else hkv
        main = [pool(B_ * max_pages, heads, s) for s in (1, 2)]
        side = [pool(B_ * ring, 1, s) for s in (3, 4)] if two_way else [None, None]
        stats = torch.randn((B_ * max_pages, heads, page // logical, 2, 128), generator=torch.Generator().manual_seed(5)).to(dtype).to(dev)
        kv = L.PagedKV(main[0], main[1], stats, table, start, pool_heads=2 if two_way else 0, k_pool_stream=side[0],
                       v_pool_stream=side[1], ring_table=ring_table if two_way else None, kv_bits=kv_bits)
        before = main[0].clone()
        L.lserve_append_kv(desc, kv, k, v, cu, start, bound)
        torch.cuda.synchronize()
        assert not torch.equal(before.view(torch.uint8), main[0].view(torch.uint8))
        results.append([t.view(torch.uint8) for t in main + side + [stats] if t is not None])
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_quantiser_codes_on_and_next_to_every_tie(dtype, bits):
    """Rows whose quotients fall on, just below and just above halves, over scales from subnormal to sixteen, and a
    constant row: the oracle's bytes."""
    L = _lib()
    dev = torch.device("cuda:0")
    top = 2 ** bits - 1
    g = torch.Generator().manual_seed(11)
    n = 640
    rows = torch.empty((n, 128), dtype=torch.float64)
    for r in range(n):
        scale = float(np.float16(2.0 ** (-24 + 28 * (r % 64) / 64)))
        zero = float(np.float16((r % 7 - 3) * scale * top))
        half = torch.randint(0, top, (128,), generator=g).double() + 0.5
        rows[r] = zero + scale * (half + (r % 5 - 2) * 2.0 ** -12 * torch.rand(128, generator=g).double())
        rows[r, 0], rows[r, 1] = zero, zero + scale * top
    rows[5] = 1.25
    x = rows.to(dtype)
    k = x.reshape(n, 1, 128).to(dev)
    pages = n // 64
    kv = L.PagedKV(torch.zeros((pages, 1, 64 * 128 * bits // 8 + 256), dtype=torch.uint8, device=dev),
                   torch.zeros((pages, 1, 64 * 128 * bits // 8 + 256), dtype=torch.uint8, device=dev),
                   torch.zeros((pages, 1, 4, 2, 128), dtype=dtype, device=dev),
                   torch.arange(pages, dtype=torch.int32, device=dev).reshape(1, -1), torch.tensor([n], dtype=torch.int32, device=dev),
                   kv_bits=bits)
    desc = L.AttnDesc(1, 1, [0], dtype=dtype)
    L.lserve_append_kv(desc, kv, k, k, torch.tensor([0, n], dtype=torch.int32, device=dev),
                       torch.zeros(1, dtype=torch.int32, device=dev), n)
    torch.cuda.synchronize()
    from test_gpu_quant import _write_rows
    ref = torch.zeros_like(kv.k_pool, device="cpu")
    _write_rows(ref, np.arange(n) // 64, 0, np.arange(n) % 64, x, bits)
    assert torch.equal(kv.k_pool.cpu(), ref) and torch.equal(kv.v_pool.cpu(), ref)


@pytest.mark.parametrize("kv_bits", [16, 8, 4])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5, 8])
def test_lists_cut_into_many_pieces(group, kv_bits):
    """One sequence, every page of it listed: up to 65 entries per list in as many ranges (or half as many), folded by all
    threads in parts; and a sequence whose pages past the selection outgrow the list."""
    L = _lib()
    dev = torch.device("cuda:0")
    w = Workload(name="pieces", batch=1, num_q_heads=2 * group, num_kv_heads=2, dtype="fp16", streaming_kv_heads=(0,),
                 sink_tokens=64, local_tokens=192, budget_tokens=4096, lengths=(4200,), decode_steps=1, seed=61 + group)
    inp = make_decode_inputs(w)
    for length, selected in ((4161, 64), (900, 14), (4000, 60), (577, 9)):
        seq = torch.tensor([length], dtype=torch.int32)
        P = -(-length // 64)
        sel = torch.full((1, 2, 64), -1, dtype=torch.int32)
        sel[0, 1, :selected] = torch.arange(selected, dtype=torch.int32)
        cnt = torch.tensor([[0, selected]], dtype=torch.int32)
        ssl = torch.tensor([min(length, selected * 64)], dtype=torch.int32)  # the pages after it were created since
        assert P >= selected
        stats = torch.zeros((inp.k_pool.shape[0], 2, 4, 2, 128), dtype=torch.float16, device=dev)
        table = inp.page_table.to(dev)
        desc = L.AttnDesc(w.num_q_heads, 2, w.streaming_flags(), dtype=torch.float16, sink_tokens=64, local_tokens=192)
        if kv_bits == 16:
            kv = L.PagedKV(inp.k_pool.to(dev), inp.v_pool.to(dev), stats, table, seq.to(dev))
        else:
            shape = (inp.k_pool.shape[0], 2, 64 * 128 * kv_bits // 8 + 256)
            kv = L.PagedKV(torch.zeros(shape, dtype=torch.uint8, device=dev), torch.zeros(shape, dtype=torch.uint8, device=dev),
                           stats, table, seq.to(dev), kv_bits=kv_bits)
            tok = torch.arange(4200)
            phys = inp.page_table[0].long()[tok // 64]
            L.lserve_append_kv(desc, kv, inp.k_pool[phys, :, tok % 64].contiguous().to(dev),
                               inp.v_pool[phys, :, tok % 64].contiguous().to(dev),
                               torch.tensor([0, 4200], dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int32, device=dev), 4200)
        ws = torch.zeros((L.lserve_workspace_bytes(L.LSERVE_CALL_SPARSE_DECODE, desc, 1, table.shape[1], 64, 0),),
                         dtype=torch.uint8, device=dev)
        outs = []
        for _ in range(2):  # the second call finds the arrival counters as the first left them
            out = torch.full((1, w.num_q_heads, 128), float("nan"), dtype=torch.float16, device=dev)
            L.lserve_sparse_decode(desc, kv, inp.q[0].to(dev), sel.to(dev), cnt.to(dev), ssl.to(dev), out, None, ws)
            outs.append(out)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1])
        if kv_bits == 16:
            ref, _ = oracle.sparse_decode(inp.q[0], inp.k_pool, inp.v_pool, inp.page_table, seq, sel.numpy(), cnt.numpy(),
                                          ssl.numpy(), w.streaming_flags(), 64, 192)
        else:
            from test_gpu_quant import _values
            ref, _ = oracle.sparse_decode_values(inp.q[0], _values(kv.k_pool.cpu(), kv_bits), _values(kv.v_pool.cpu(), kv_bits),
                                                 inp.page_table, seq, sel.numpy(), cnt.numpy(), ssl.numpy(),
                                                 w.streaming_flags(), 64, 192)
        assert_attention_close(outs[0], np.asarray(ref).reshape(1, w.num_q_heads, 128), f"pieces {group} {kv_bits} {length}")


def test_covered_sequences_take_no_scores_but_their_statistics_are_brought_up_to_date():
    """A budget over the whole context selects every page; without a score array only stale statistics are rebuilt."""
    L = _lib()
    dev = torch.device("cuda:0")
    lengths = (700, 64, 130, 3000)
    w = Workload(name="cov", batch=4, num_q_heads=4, num_kv_heads=2, dtype="fp16", streaming_kv_heads=(), lengths=lengths,
                 decode_steps=1, budget_tokens=1024, seed=71)
    inp = make_decode_inputs(w)
    table, seq = inp.page_table.to(dev), torch.tensor(lengths, dtype=torch.int32, device=dev)
    desc = L.AttnDesc(4, 2, [0, 0], dtype=torch.float16)
    k, v = inp.k_pool.to(dev), inp.v_pool.to(dev)
    full = torch.zeros((k.shape[0], 2, 4, 2, 128), dtype=torch.float16, device=dev)
    L.lserve_build_page_stats(desc, L.PagedKV(k, v, full, table, seq), None, 0)
    valid = torch.tensor([0, 63, 0, 2900], dtype=torch.int32, device=dev)
    stats = torch.zeros_like(full)
    for b, n in enumerate((0, 63, 0, 2900)):  # what is current before the call: whole logical pages below `valid`
        for lp in range(n // 16):
            phys = int(inp.page_table[b, lp // 4])
            stats[phys, :, lp % 4] = full[phys, :, lp % 4]
    picked = []
    for scores in (None, torch.empty((4, 2, table.shape[1]), device=dev)):
        s = stats.clone()
        kv = L.PagedKV(k, v, s, table, seq)
        sel = torch.full((4, 2, 16), -7, dtype=torch.int32, device=dev)
        cnt, ssl = torch.zeros((4, 2), dtype=torch.int32, device=dev), torch.zeros(4, dtype=torch.int32, device=dev)
        ws = torch.empty((L.lserve_workspace_bytes(L.LSERVE_CALL_SELECT_PAGES, desc, 4, table.shape[1], 16, 0),),
                         dtype=torch.uint8, device=dev)
        L.lserve_select_pages(desc, kv, inp.q[0].to(dev), 1024, sel, cnt, ssl, scores, ws, stats_valid_len=valid)
        torch.cuda.synchronize()
        assert torch.equal(s, full)
        picked.append((sel, cnt, ssl))
    assert all(torch.equal(a, b) for a, b in zip(*picked))
    assert cnt[:3, 0].tolist() == [11, 1, 3] and cnt[3].tolist() == [16, 16]


@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("dtype,kv_bits,span", [(torch.float16, 4, 20000.0), (torch.float16, 4, 65504.0), (torch.bfloat16, 4, 60000.0),
                                                (torch.bfloat16, 8, 3e5), (torch.bfloat16, 8, 6e6)])
def test_quantised_decode_over_value_rows_of_any_scale(dtype, kv_bits, span, group):
    """A few value rows spanning `span` either way among rows of N(0, 1), anywhere in the list: their scales times the weights
    times the factor that suits the other rows are beyond fp16."""
    L = _lib()
    dev = torch.device("cuda:0")
    n, heads = 3000, 2
    g = torch.Generator().manual_seed(97 + group)
    k = torch.randn((n, heads, 128), generator=g)
    v = torch.randn((n, heads, 128), generator=g)
    loud = torch.randint(0, n, (40,), generator=g)
    k[loud] *= 2.5  # and they take the largest weights
    v[loud] = (torch.rand((40, heads, 128), generator=g) * 2 - 1) * span
    k, v = k.to(dtype), v.to(dtype)
    q = torch.randn((1, heads * group, 128), generator=g).to(dtype)
    pages = -(-n // 64)
    shape = (pages, heads, 64 * 128 * kv_bits // 8 + 256)
    seq = torch.tensor([n], dtype=torch.int32)
    kv = L.PagedKV(torch.zeros(shape, dtype=torch.uint8, device=dev), torch.zeros(shape, dtype=torch.uint8, device=dev),
                   torch.zeros((pages, heads, 4, 2, 128), dtype=dtype, device=dev),
                   torch.arange(pages, dtype=torch.int32, device=dev).reshape(1, -1), seq.to(dev), kv_bits=kv_bits)
    desc = L.AttnDesc(heads * group, heads, [0, 0], dtype=dtype)
    L.lserve_append_kv(desc, kv, k.to(dev), v.to(dev), torch.tensor([0, n], dtype=torch.int32, device=dev),
                       torch.zeros(1, dtype=torch.int32, device=dev), n)
    sel = torch.arange(pages, dtype=torch.int32).repeat(1, heads, 1)
    cnt = torch.full((1, heads), pages, dtype=torch.int32)
    out = torch.full((1, heads * group, 128), float("nan"), dtype=dtype, device=dev)
    L.lserve_sparse_decode_noalloc(desc, kv, q.to(dev), sel.to(dev), cnt.to(dev), seq.to(dev), out, None)
    torch.cuda.synchronize()
    from test_gpu_quant import _values
    ref, _ = oracle.sparse_decode_values(q, _values(kv.k_pool.cpu(), kv_bits), _values(kv.v_pool.cpu(), kv_bits),
                                         torch.arange(pages, dtype=torch.int32).reshape(1, -1), seq, sel.numpy(), cnt.numpy(),
                                         seq.numpy(), [0, 0], 64, 64)
    ref = np.asarray(ref).reshape(heads * group, 128)
    got = out.double().cpu().numpy().reshape(heads * group, 128)
    assert np.isfinite(got).all()
    # weights are rounded to fp16 (2^-11 relative), outputs to their type (2^-11 or 2^-8): the row bound of the other tests
    rel = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert rel.max() <= 1e-2, rel.max()
