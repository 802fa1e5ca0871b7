"""Softmax of prefill relative to a reference that is only moved when weights grow large: scores that climb, jump and fall along
a sequence, rows without a reference, rows that are not numbers; sampled rows against the oracle.  Prompts, listed masks in every walk, and
chunks over pages of every width, whole, in pieces and over expanded pages.

Scaled keys leave logits of up to some hundreds, whose fp32 products are exact to 1e-4 at worst, so the bounds of the other prefill
tests hold."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_chunk_expand as expand
import test_gpu_chunk_pieces as pieces
import test_gpu_masked_shared as masked
import test_gpu_paged_shapes as paged
import test_gpu_prefill_shapes as shapes
from workloads import Workload, make_prefill_inputs

from parity import LSE_TOL_PREFILL, assert_attention_close, assert_lse_close

pytestmark = pytest.mark.gpu

SHAPES = [(64, 8, (1100, 77, 640)),    # half workgroups
          (32, 8, (1500,)),            # two slices
          (8, 8, (4500, 1)),           # four
          (16, 8, (12001, 64)),        # whole workgroups, long walks
          (8, 2, (51, 7, 33))]         # and of one tile


def _factor(pattern, n):
    t = np.arange(n)
    if pattern == "climb":        # past the largest weight, tile after tile
        return 0.05 + 12.0 * t / n
    if pattern == "jumps":        # one loud key among 150, each louder than the last (a row may go from weight 1 to 2^200 at once)
        return np.where(t % 150 == 149, 4.0 + 16.0 * t / n, 1.0)
    if pattern == "island":       # the loud ones lie together, in one piece of a cut walk
        return np.where((t > n // 3) & (t < n // 3 + 200), 12.0, 0.5)
    return 12.0 / (1 + t / 40.0)  # falls: the first keys are the loudest


def _run(w, lengths, pin):
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    desc = L.AttnDesc(w.num_q_heads, w.num_kv_heads, w.streaming_flags(), dtype=w.torch_dtype,
                      sink_tokens=w.sink_tokens, local_tokens=w.local_tokens)
    q, k, v, cu = pin.q.to(dev), pin.k.to(dev), pin.v.to(dev), pin.cu_seqlens.to(dev)
    out = torch.full_like(q, float("nan"))
    lse = torch.full((w.num_q_heads, q.shape[0]), float("nan"), dtype=torch.float32, device=dev)
    L.lserve_sparse_prefill(desc, q, k, v, cu, max(lengths), out, lse)
    torch.cuda.synchronize()
    return out, lse


def _check(w, pin, out, lse, tok, what):
    heads = w.num_q_heads
    t, h = np.repeat(tok, heads).astype(np.int32), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.sparse_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64, w.sink_tokens,
                                              w.local_tokens, t, h)
    at = torch.as_tensor(tok).long().to(out.device)
    assert_attention_close(out[at], ref.reshape(len(tok), heads, -1), what)
    assert_lse_close(lse.t()[at].contiguous(), lse_ref.reshape(len(tok), heads), what + " lse", LSE_TOL_PREFILL[w.dtype])


def _layer(heads, kv_heads, lengths, dtype):
    return Workload(name="ref", batch=len(lengths), num_q_heads=heads, num_kv_heads=kv_heads, dtype=dtype,
                    streaming_kv_heads=tuple(range(kv_heads // 2)), sink_tokens=64, local_tokens=192, seed=91)


def _rows(lengths, first=0):
    rng, at, tok = np.random.default_rng(3), 0, []
    for n in lengths:
        if n > first:
            tok += sorted({at + first, at + n - 1} | {at + int(r) for r in rng.integers(first, n, 20)})
        at += n
    return np.asarray(tok)


def _louder(pattern):
    """make_prefill_inputs with the keys of every sequence scaled along it."""
    def make(w, lengths):
        pin = make_prefill_inputs(w, lengths=lengths)
        f = np.concatenate([_factor(pattern, n) for n in lengths])
        pin.k.copy_((pin.k.float() * torch.from_numpy(f).float()[:, None, None]).to(pin.k.dtype))
        return pin
    return make


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("pattern", ["climb", "jumps", "falls"])
@pytest.mark.parametrize("heads,kv_heads,lengths", SHAPES)
def test_scores_that_move(dtype, pattern, heads, kv_heads, lengths):
    w = _layer(heads, kv_heads, lengths, dtype)
    pin = _louder(pattern)(w, lengths)
    out, lse = _run(w, lengths, pin)
    _check(w, pin, out, lse, _rows(lengths), f"{pattern} {dtype} {heads}/{kv_heads}")


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,lengths", SHAPES[:4])
def test_rows_whose_first_tile_is_minus_infinity(dtype, heads, kv_heads, lengths):
    """Rows past the first tile take nothing from it, and their reference from the first tile that has one."""
    w = _layer(heads, kv_heads, lengths, dtype)
    pin = make_prefill_inputs(w, lengths=lengths)
    pin.q[:, :, 5] = 1.0
    at = 0
    for n in lengths:
        pin.k[at:at + min(n, 64), :, 5] = -float("inf")
        at += n
    out, lse = _run(w, lengths, pin)
    _check(w, pin, out, lse, _rows(lengths, first=64), f"-inf {dtype} {heads}/{kv_heads}")


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("heads,kv_heads,lengths", SHAPES)
def test_a_query_that_is_not_a_number_keeps_to_itself(dtype, value, heads, kv_heads, lengths):
    """Row sums of two queries come out of one column of a matrix product."""
    w = _layer(heads, kv_heads, lengths, dtype)
    pin = make_prefill_inputs(w, lengths=lengths)
    bad = np.arange(5, sum(lengths), 37)
    good = np.setdiff1d(np.concatenate([bad - 16, bad + 16, _rows(lengths)]), bad)
    good = good[(good >= 0) & (good < sum(lengths))][:120]
    clean = pin.q.clone()
    pin.q[torch.from_numpy(bad)] = value
    out, lse = _run(w, lengths, pin)
    pin.q.copy_(clean)
    assert torch.isnan(out[torch.from_numpy(bad).to(out.device)]).all()
    _check(w, pin, out, lse, good, f"{value} {dtype} {heads}/{kv_heads}")


WALKS = [(32, 8, (1500, 333), ("few", "other"), [-1] * 16 + [0, 1, 0, 1] * 4, shapes.HALVES),
         (24, 8, (2500, 70), ("few",), [-1] * 7 + [0] * 17, shapes.SLICES),
         (32, 8, (3001, 500), ("most", "holes", "all"), [h % 4 - 1 for h in range(32)], shapes.MERGED)]


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("pattern", ["climb", "jumps", "falls"])
@pytest.mark.parametrize("walk", range(3))
def test_scores_that_move_under_listed_masks(dtype, pattern, walk, monkeypatch):
    monkeypatch.setattr(shapes, "make_prefill_inputs", _louder(pattern))
    masked.test_two_heads_to_a_row(dtype, *WALKS[walk])


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,lengths,dense,walk", [
    (32, 8, (2600,), False, shapes.HALVES), (24, 8, (2500, 300), False, shapes.SLICES), (32, 8, (5000, 500), True, shapes.MERGED)])
def test_rows_of_listed_masks_whose_first_tile_is_minus_infinity(dtype, heads, kv_heads, lengths, dense, walk, monkeypatch):
    """The first tile is kept by all rows, and the second by few: references come late, and at another tile in every row."""
    def make(w, lengths):
        pin = make_prefill_inputs(w, lengths=lengths)
        pin.q[:, :, 5] = 1.0
        at = 0
        for n in lengths:
            pin.k[at:at + 64, :, 5] = -float("inf")
            at += n
        return pin
    monkeypatch.setattr(shapes, "make_prefill_inputs", make)
    w = Workload(name="ref", batch=len(lengths), num_q_heads=heads, num_kv_heads=kv_heads, dtype=dtype,
                 streaming_kv_heads=tuple(range(kv_heads // 2)), sink_tokens=64, local_tokens=256, seed=91)
    masks = [lambda b, i: [j for j in range(i + 1) if j in (0, i) or ((7 * j + 3 * i) % (9 if dense else 5) == 0) != dense],
             lambda b, i: [j for j in range(i + 1) if j in (0, i) or ((j + i) % 7 == 0) != dense]]
    head_mask = [h % 2 for h in range(heads)]
    pin, out, lse, (qts, rp, cl, rows) = shapes._run(w, lengths, masks, head_mask, walk=walk)
    tok = _rows(lengths, first=64)
    t, h = np.repeat(tok, heads).astype(np.int32), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.block_mask_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64, w.sink_tokens,
                                                  w.local_tokens, head_mask, qts, rp, cl, rows, t, h)
    shapes._check(w, lengths, pin, out, lse, ref, lse_ref, tok, f"masked -inf {dtype} {heads}/{kv_heads}")


def _rounded_history(dtype):
    """What a cache holds as the kernels see it: dequantised values rounded to the layer's type (of loud keys the rounding shows)."""
    exact = paged._history
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    return lambda *a: [torch.from_numpy(x).to(dt).double().numpy() for x in exact(*a)]


CHUNKS = [(32, 8, (101, 333), (1500, 1500), {16: None, 8: None, 4: None}),  # half workgroups
          (12, 4, (64, 901, 3000), (0, 65, 130), {16: None, 8: None, 4: None})]  # four slices, two over quantised pages


@pytest.mark.parametrize("dtype,bits,two_way", [("fp16", 16, False), ("bf16", 16, True), ("fp16", 8, True), ("bf16", 4, False)])
@pytest.mark.parametrize("pattern", ["climb", "jumps", "falls"])
@pytest.mark.parametrize("case", range(len(CHUNKS)))
def test_scores_that_move_in_chunks(case, pattern, dtype, bits, two_way, monkeypatch):
    monkeypatch.setattr(paged, "make_prefill_inputs", _louder(pattern))
    monkeypatch.setattr(paged, "_history", _rounded_history(dtype))
    monkeypatch.setattr(paged, "CASES", CHUNKS)
    paged.test_chunks_in_every_launch_shape(case, dtype, bits, two_way)


@pytest.mark.parametrize("dtype,bits,two_way", [("fp16", 16, False), ("bf16", 16, True), ("bf16", 8, False), ("fp16", 4, True)])
@pytest.mark.parametrize("pattern", ["climb", "jumps", "falls", "island"])
@pytest.mark.parametrize("case", [2, 4])
def test_scores_that_move_in_pieces(case, pattern, dtype, bits, two_way, monkeypatch):
    """References of a block's pieces lie far apart.  (That walks are cut, and streaming heads beside the fold, is asserted there.)"""
    monkeypatch.setattr(paged, "make_prefill_inputs", _louder(pattern))
    monkeypatch.setattr(paged, "_history", _rounded_history(dtype))
    pieces.test_chunks_in_pieces(case, dtype, bits, two_way, monkeypatch)


@pytest.mark.parametrize("dtype,bits", [("bf16", 8), ("fp16", 4)])
@pytest.mark.parametrize("pattern", ["climb", "island"])
@pytest.mark.parametrize("case", [1, 7])
def test_scores_that_move_over_expanded_pages(case, pattern, dtype, bits, monkeypatch):
    monkeypatch.setattr(paged, "make_prefill_inputs", _louder(pattern))
    monkeypatch.setattr(paged, "_history", _rounded_history(dtype))
    expand.test_chunks_over_expanded_pages(case, dtype, bits, False, monkeypatch)
