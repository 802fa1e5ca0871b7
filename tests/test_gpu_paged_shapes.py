"""Chunks over pages in every shape the host chooses for them (one, two and four key slices, heads or query tiles as the units
of a workgroup, streaming heads folded or in units of their own, blocks in order or per sequence), over 16-, 8- and 4-bit
pages, one pool and the two-way cache: sampled rows against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload, make_prefill_inputs

from parity import LSE_TOL_PREFILL, assert_attention_close, assert_lse_close
from test_gpu_chunk_prefill import LSE_TOL_QUANT_HISTORY
from test_gpu_quant import _values

pytestmark = pytest.mark.gpu

NP, SINK, LOCAL = 64, 64, 192


def _history(kv, bits, table, ring_table, hist, streaming, s_pages, w_pages, hkv):
    """float64 [B, max hist, Hkv, D] x 2: what the cache holds for every history position, NaN where it holds nothing."""
    def pools(t):
        if t is None:
            return None
        return t.cpu().double().numpy() if bits == 16 else _values(t.cpu(), bits)
    main, ring = [pools(kv.k_pool), pools(kv.v_pool)], [pools(kv.k_pool_stream), pools(kv.v_pool_stream)]
    dense = [h for h in range(hkv) if h not in streaming]
    out = [np.full((len(hist), max(max(hist), 1), hkv, 128), np.nan) for _ in range(2)]
    for b, S in enumerate(hist):
        u = np.arange(S)
        p, t = u // NP, u % NP
        P = -(-S // NP)
        for hk in range(hkv):
            for side in range(2):
                if ring[0] is not None and hk in streaming:
                    kept = (p < s_pages) | (p >= P - w_pages)
                    slot = np.where(p < s_pages, p, s_pages + (p - s_pages) % w_pages)
                    rows = ring[side][ring_table[b].numpy()[slot], streaming.index(hk), t]
                    out[side][b, :S, hk] = np.where(kept[:, None], rows, np.nan)
                else:
                    rank = dense.index(hk) if main[side].shape[1] != hkv else hk
                    out[side][b, :S, hk] = main[side][table[b].numpy()[p], rank, t]
    return out


def _sample(fresh, per_seq, seed):
    rng = np.random.default_rng(seed)
    tok, at = [], 0
    for n in fresh:
        if n:
            tok += [at + r for r in sorted({0, n - 1, min(63, n - 1), min(64, n - 1), n // 2} | set(rng.integers(0, n, per_seq).tolist()))]
        at += n
    return np.asarray(tok, dtype=np.int32)


# heads, KV heads, history, new tokens, {bits: (slices, dense folded, streaming folded, units are query tiles)}; "half": the launch over 16
# bits is by half workgroups; "expand": that over quantised pages goes over expanded ones
CASES = [
    (32, 8, (101, 333), (1500, 1500), {16: (1, 0, 0, 0), 8: (1, 0, 0, 0), 4: (1, 0, 0, 0), "half": 1, "expand": 0}),
    # whole workgroups in one slice: four heads to one, and four tiles
    (32, 8, (4400, 4100), (2500, 2600), {16: (1, 0, 0, 0), 8: (1, 0, 0, 0), 4: (1, 0, 0, 0), "half": 0, "expand": 1}),
    (24, 8, (6001, 6000), (1500, 2000), {16: (1, 0, 0, 0), 8: (1, 0, 0, 0), 4: (1, 0, 0, 0), "half": 0, "expand": 1}),
    (32, 8, (1500,), (4096,), {16: (2, 1, 0, 0), 8: (1, 0, 0, 1), 4: (1, 0, 0, 1)}),
    (32, 8, (1500, 37), (700, 2200), {16: (2, 1, 0, 0), 8: (2, 1, 0, 0), 4: (2, 1, 0, 0)}),
    (32, 8, (101, 0), (300, 1200), {16: (2, 1, 1, 0), 8: (2, 1, 1, 0), 4: (2, 1, 1, 0)}),
    (32, 8, (101,), (600,), {16: (2, 1, 1, 1), 8: (2, 1, 1, 1), 4: (2, 1, 1, 1)}),
    (12, 4, (64, 901, 3000), (0, 65, 130), {16: (4, 1, 1, 0), 8: (2, 1, 1, 1), 4: (2, 1, 1, 1)}),
    # several sequences to a lane, idle ones among them; more than are dealt out in order
    (8, 2, tuple(5 + 13 * i for i in range(67)), tuple((7 * i) % 131 for i in range(67)), {16: None, 8: None, 4: None}),
    (4, 2, tuple((29 * i) % 211 for i in range(270)), tuple((7 * i) % 67 for i in range(270)), {16: None, 8: None, 4: None}),
]


@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("dtype,bits", [("fp16", 16), ("bf16", 16), ("fp16", 8), ("bf16", 8), ("fp16", 4), ("bf16", 4)])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_chunks_in_every_launch_shape(case, dtype, bits, two_way):
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    heads, hkv, hist, fresh, shapes = CASES[case]
    streaming = tuple(range(hkv // 2))
    B, lengths = len(hist), tuple(h + n for h, n in zip(hist, fresh))
    w = Workload(name="paged", batch=B, num_q_heads=heads, num_kv_heads=hkv, dtype=dtype, streaming_kv_heads=streaming,
                 sink_tokens=SINK, local_tokens=LOCAL, seed=91 + case)
    pin = make_prefill_inputs(w, lengths=lengths)
    pages = max(-(-n // NP) for n in lengths)
    desc = L.AttnDesc(heads, hkv, w.streaming_flags(), dtype=w.torch_dtype, sink_tokens=SINK, local_tokens=LOCAL)
    if shapes[bits] is not None:
        assert L.lserve_probe_prefill_shape(desc, B, sum(fresh), max(fresh), pages, bits) == shapes[bits]
    if "half" in shapes:
        plan = L.lserve_probe_prefill_plan(desc, B, sum(fresh), max(fresh), pages, bits)
        assert plan["half"] == (shapes["half"] and bits == 16) and plan["expand"] == (shapes["expand"] and bits != 16)
    s_pages, w_pages = SINK // NP, LOCAL // NP
    g = torch.Generator().manual_seed(case)
    table = torch.randperm(B * pages, generator=g).to(torch.int32).reshape(B, pages)
    ring_table = torch.randperm(B * (s_pages + w_pages), generator=g).to(torch.int32).reshape(B, -1)

    def pool(n, h):  # what was never written is not a number, as rows or as scales
        if bits == 16:
            return torch.full((n, h, NP, 128), float("nan"), dtype=w.torch_dtype, device=dev)
        return torch.full((n, h, NP * 128 * bits // 8 + 256), 0xff, dtype=torch.uint8, device=dev)
    main_heads = hkv - len(streaming) if two_way else hkv
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    seq = i32([max(h, 1) for h in hist])
    kv = L.PagedKV(pool(B * pages, main_heads), pool(B * pages, main_heads),
                   torch.zeros((B * pages, main_heads, 4, 2, 128), dtype=w.torch_dtype, device=dev), table.to(dev), seq, kv_bits=bits)
    if two_way:
        n = ring_table.numel()
        kv.pool_heads, kv.ring_table = main_heads, ring_table.to(dev)
        kv.k_pool_stream, kv.v_pool_stream = pool(n, len(streaming)), pool(n, len(streaming))
    cut = lambda t, past: torch.cat([t[int(c) + (0 if past else h):int(c) + (h if past else h + n)]
                                     for c, h, n in zip(pin.cu_seqlens, hist, fresh)]).contiguous()
    cu = lambda xs: np.concatenate([[0], np.cumsum(xs)]).astype(np.int32)
    L.lserve_append_kv(desc, kv, cut(pin.k, True).to(dev), cut(pin.v, True).to(dev), i32(cu(hist)), i32([0] * B), max(hist))
    kv.seq_lens = i32(list(hist))
    q, k, v = cut(pin.q, False), cut(pin.k, False), cut(pin.v, False)
    out = torch.full((len(q), heads, 128), float("nan"), dtype=w.torch_dtype, device=dev)
    lse = torch.full((heads, len(q)), float("nan"), dtype=torch.float32, device=dev)
    L.lserve_sparse_prefill_chunk(desc, kv, q.to(dev), k.to(dev), v.to(dev), i32(cu(fresh)), max(fresh), out, lse)
    torch.cuda.synchronize()
    assert not torch.isnan(out).any() and not torch.isnan(lse).any()
    tok = _sample(fresh, 1 if B > 99 else 3 if B > 8 else 12, case)
    kh, vh = _history(kv, bits, table, ring_table, hist, streaming, s_pages, w_pages, hkv)
    t, h = np.repeat(tok, heads), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.chunk_prefill_rows(q, k, v, kh, vh, np.asarray(hist, np.int32), cu(fresh), w.streaming_flags(), NP,
                                             SINK, LOCAL, t, h)
    at = torch.from_numpy(tok).long().to(dev)
    what = f"chunk {case} {dtype} {bits} two_way={two_way}"
    assert_attention_close(out[at], ref.reshape(len(tok), heads, -1), what)
    tol = (LSE_TOL_PREFILL if bits == 16 else LSE_TOL_QUANT_HISTORY)[dtype]
    assert_lse_close(lse.t()[at].contiguous(), lse_ref.reshape(len(tok), heads), what + " lse", tol)
