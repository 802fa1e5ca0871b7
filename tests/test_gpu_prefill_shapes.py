"""Prefill of prompts in every launch shape the host chooses (one, two and four key slices, heads or query tiles as the units
of a workgroup, blocks in order over the batch or per sequence), sampled rows against the oracle.  Chunks over pages:
test_gpu_paged_shapes.py."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload, make_prefill_inputs

from parity import LSE_TOL_PREFILL, assert_attention_close, assert_lse_close

pytestmark = pytest.mark.gpu

MERGED, SLICES, HALVES = 0, 1, 2  # of lserve_probe_mask_walk


def _run(w, lengths, mask=None, head_mask=None, past_diagonal=0, walk=None):
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    pin = make_prefill_inputs(w, lengths=lengths)
    desc = L.AttnDesc(w.num_q_heads, w.num_kv_heads, w.streaming_flags(), dtype=w.torch_dtype,
                      sink_tokens=w.sink_tokens, local_tokens=w.local_tokens)
    q, k, v, cu = pin.q.to(dev), pin.k.to(dev), pin.v.to(dev), pin.cu_seqlens.to(dev)
    out = torch.full_like(q, float("nan"))
    lse = torch.full((w.num_q_heads, q.shape[0]), float("nan"), dtype=torch.float32, device=dev)
    if mask is None:
        L.lserve_sparse_prefill(desc, q, k, v, cu, max(lengths), out, lse)
        csr = None
    else:
        from helpers import block_mask_csr
        qts, rp, cl, rows = csr = block_mask_csr(mask, lengths)
        if past_diagonal:  # entries above a row's own tile, to be ignored: the same for both sides but for these
            tile = np.concatenate([np.arange(b - a) for a, b in zip(qts[:-1], qts[1:])] * len(mask))
            last = np.concatenate([np.full(b - a, b - a) for a, b in zip(qts[:-1], qts[1:])] * len(mask))
            more = [list(cl[rp[r]:rp[r + 1]]) + list(range(tile[r] + 1, min(tile[r] + past_diagonal, last[r])))
                    for r in range(len(tile))]
            rp = np.concatenate([[0], np.cumsum([len(x) for x in more])])
            cl = np.concatenate(more)
        i32 = lambda a: torch.as_tensor(np.asarray(a, dtype=np.int32)).to(dev)
        bm = L.BlockMask(i32(head_mask), i32(qts), i32(rp), i32(cl), len(mask), rows)
        if walk is not None:
            assert L.lserve_probe_mask_walk(desc, len(lengths), q.shape[0], max(lengths), len(mask), rows, len(cl)) == walk
        need = L.lserve_masked_prefill_workspace_bytes(desc, len(lengths), q.shape[0], max(lengths), len(mask), len(cl))
        ws = torch.empty((need,), dtype=torch.uint8, device=dev)
        L.lserve_sparse_prefill_masked(desc, bm, q, k, v, cu, max(lengths), out, lse, ws)
    torch.cuda.synchronize()
    assert not torch.isnan(out).any() and not torch.isnan(lse).any()
    return pin, out, lse, csr


def _sample(lengths, per_seq, seed):
    """First, last and random rows of every sequence, tile edges among them."""
    rng = np.random.default_rng(seed)
    tok, at = [], 0
    for n in lengths:
        rows = {0, n - 1, min(63, n - 1), min(64, n - 1), (n - 1) // 64 * 64} | set(rng.integers(0, n, per_seq).tolist())
        tok += [at + r for r in sorted(rows)]
        at += n
    return np.asarray(tok, dtype=np.int32)


def _check(w, lengths, pin, out, lse, ref, lse_ref, tok, what):
    H = w.num_q_heads
    got = out[torch.from_numpy(tok).long().to(out.device)]
    assert_attention_close(got, ref.reshape(len(tok), H, -1), what)
    got_lse = lse.t()[torch.from_numpy(tok).long().to(out.device)].contiguous()
    assert_lse_close(got_lse, lse_ref.reshape(len(tok), H), what + " lse", LSE_TOL_PREFILL[w.dtype])


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,lengths,shape,half", [  # (slices, dense folded, streaming folded, units are query tiles)
    (8, 2, (65,), (1, 0, 0, 1), 1),                    # walks of one or two tiles
    (32, 8, (1500,), (2, 1, 1, 1), 0),
    (32, 8, (2047,), (2, 1, 1, 0), 0),                 # two slices, streaming heads folded too
    (32, 8, (4097,), (2, 1, 0, 0), 0),                 # streaming heads in units of their own
    (8, 8, (4500, 1), (4, 1, 1, 0), 0),                # no groups; one-token sequence
    (12, 4, (3000, 700), (4, 1, 1, 0), 0),             # three heads per group: neither two nor four divide it
    (16, 4, (1000, 1000, 1000), (2, 1, 0, 0), 0),      # equal lengths are not searched
    (12, 2, (1500, 333, 64), (4, 1, 1, 0), 0),         # six: two heads and two query tiles, where four units share a walk
    # half workgroups
    (64, 8, (1100, 77, 640), (1, 0, 0, 0), 1),         # eight: heads of a group in several workgroups
    (8, 2, tuple(3 + 17 * i for i in range(64)), (1, 0, 0, 0), 1),  # one sequence to every lane
    (8, 2, tuple(5 + 16 * i for i in range(67)), (1, 0, 0, 0), 1),  # two to some
    (4, 2, tuple(1 + (37 * i) % 400 for i in range(200)), (1, 0, 0, 0), 1),  # four to some
    (4, 2, (130,) * 200, (1, 0, 0, 0), 1),                                   # and all alike
    (4, 2, tuple(1 + (37 * i) % 300 for i in range(256)), (1, 0, 0, 0), 1),  # the largest batch dealt out in order
    (4, 2, tuple(1 + (37 * i) % 300 for i in range(257)), (1, 0, 0, 0), 1),  # a batch beyond that
    # whole ones in one slice
    (32, 8, (12001, 333), (1, 0, 0, 0), 0),            # four heads to a workgroup
    (16, 4, (12001, 333), (1, 0, 0, 1), 0),            # four tiles of one head
    (24, 8, (9001, 9500), (1, 0, 0, 0), 0),            # no two heads of three: four tiles
    (16, 8, (12001, 5000, 64), (1, 0, 0, 0), 0),       # two heads, two tiles
    (16, 16, (12001,), (1, 0, 0, 0), 0),               # no groups
    (64, 8, (128,) * 16, (1, 0, 0, 0), 0),             # two full rounds
    (32, 8, (231,) * 8, (1, 0, 0, 0), 0),              # one
    (32, 32, (385,) * 4, (1, 0, 0, 0), 0),
    (8, 2, (51, 7, 33), (1, 0, 0, 1), 0),              # a single tile each
])
def test_prefill_launch_shapes(dtype, heads, kv_heads, lengths, shape, half):
    w = Workload(name="ps", batch=len(lengths), num_q_heads=heads, num_kv_heads=kv_heads, dtype=dtype,
                 streaming_kv_heads=tuple(range(kv_heads // 2)), sink_tokens=64, local_tokens=192, seed=53)
    import paper_2502_14866_amd as L
    desc = L.AttnDesc(heads, kv_heads, w.streaming_flags(), dtype=w.torch_dtype, sink_tokens=64, local_tokens=192)
    assert L.lserve_probe_prefill_shape(desc, len(lengths), sum(lengths), max(lengths)) == shape
    assert L.lserve_probe_prefill_plan(desc, len(lengths), sum(lengths), max(lengths))["half"] == half
    pin, out, lse, _ = _run(w, lengths)
    tok = _sample(lengths, 1 if len(lengths) > 99 else 6 if len(lengths) > 8 else 24, 5)
    t, h = np.repeat(tok, heads), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.sparse_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64, w.sink_tokens,
                                              w.local_tokens, t, h)
    _check(w, lengths, pin, out, lse, ref, lse_ref, tok, f"prefill {dtype} {heads}/{kv_heads} {len(lengths)} sequences")


@pytest.mark.parametrize("lengths,walk", [((10300, 333), HALVES), ((2100, 64), HALVES), ((300, 129), SLICES),
                                          ((4500, 333), MERGED), ((3001, 500), MERGED)])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_masked_prefill_walks_merged_lists_and_the_callers_rows(dtype, lengths, walk):
    """Mask 0 keeps the same tiles in neighbouring rows, mask 1 others in every row, mask 2 mixes the two by block; one head
    keeps the analytic pattern; row lists go on past the diagonal and are cut there.  Lists of a third of the tiles are walked as the
    caller's rows, the smallest batch in four key slices, lists of most of them merged."""
    w = Workload(name="pm3", batch=2, num_q_heads=32, num_kv_heads=8, dtype=dtype, streaming_kv_heads=(0, 1, 2, 3),
                 sink_tokens=128, local_tokens=512, seed=59)
    dense = walk == MERGED  # keep what the others drop
    same = lambda b, i: [j for j in range(i + 1) if (j % 3 == 0) != dense or j == i]
    other = lambda b, i: [j for j in range(i + 1) if ((j + i) % 4 == 0) != dense or j == i]
    mixed = lambda b, i: same(b, i) if (i // 4) % 2 else other(b, i)
    head_mask = [-1 if h < 13 else h % 3 for h in range(32)]
    pin, out, lse, (qts, rp, cl, rows) = _run(w, lengths, [same, other, mixed], head_mask, past_diagonal=7, walk=walk)
    tok = _sample(lengths, 40, 9)
    t, h = np.repeat(tok, 32), np.tile(np.arange(32, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.block_mask_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64,
                                                  w.sink_tokens, w.local_tokens, head_mask, qts, rp, cl, rows, t, h)
    _check(w, lengths, pin, out, lse, ref, lse_ref, tok, f"masked prefill {dtype}")


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_paged_prefill_goes_by_the_stated_length_not_by_the_width_of_the_table(dtype):
    """The same cache behind a table of 32 and of 2048 pages per sequence: the launch, and so every bit, is the same."""
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    n = 2047
    w = Workload(name="width", batch=1, num_q_heads=32, num_kv_heads=8, dtype=dtype, streaming_kv_heads=(0, 1, 2, 3),
                 sink_tokens=128, local_tokens=512, seed=83)
    pin = make_prefill_inputs(w, lengths=(n,))
    desc = L.AttnDesc(32, 8, w.streaming_flags(), dtype=w.torch_dtype, sink_tokens=128, local_tokens=512)
    pool = lambda t: torch.cat([t, t[:1]]).reshape(32, 64, 8, 128).transpose(1, 2).contiguous().to(dev)
    k, v, q, cu = pool(pin.k), pool(pin.v), pin.q.to(dev), pin.cu_seqlens.to(dev)
    outs = []
    for width in (32, 2048):
        table = torch.zeros((1, width), dtype=torch.int32)
        table[0, :32] = torch.arange(32)
        kv = L.PagedKV(k, v, None, table.to(dev), torch.tensor([n], dtype=torch.int32, device=dev))
        out, lse = torch.empty_like(q), torch.empty((32, n), dtype=torch.float32, device=dev)
        L.lserve_sparse_prefill_paged(desc, kv, q, cu, n, n, out, lse, None)
        outs.append((out, lse))
    torch.cuda.synchronize()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
