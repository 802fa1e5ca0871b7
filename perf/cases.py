"""The calls whose speed counts: what a serving layer asks of the attention path, from one short sequence to the
longest prompt, each through the public entry points.

A case is a dict of plain values.  Its `kind` says which call it is:

  decode   one reuse interval of the decode loop: four steps, each writing the new token's K / V into the cache and
           attending the index table, with one selector run on the first of them (DecodeSession)
  prefill  block-sparse causal prefill of a batch of prompts (lserve_sparse_prefill)
  chunk    a chunk of new tokens over a history that is already in the paged cache (lserve_sparse_prefill_chunk)
  masked   prefill under a listed block mask for the dense heads (lserve_sparse_prefill_masked)
  append   write-back of the prompts' K / V into the pages, statistics included (lserve_append_kv)

Half of the KV heads stream (128 sink and 512 local tokens) and the other half select or attend densely, the layer
shape all decode and prefill configurations of this repository share.  K is N(0, 1) times a factor per (head, channel) as
real keys have loud channels, Q and V are N(0, 1).
"""
from __future__ import annotations

import math

import torch

import paper_2502_14866_amd.binding as B
from paper_2502_14866_amd.session import DecodeSession

D = 128
TILE = 64
SINK, LOCAL = 128, 512
STEPS = 4  # decode steps per selector run


def _case(name, kind, **kw):
    case = {"name": name, "kind": kind, "dtype": "fp16", "q_heads": 32, "kv_heads": 8, "batch": 1, "shortest": 0,
            "longest": 0, "kv_bits": 16, "two_way": False, "page": 64, "budget": 4096, "history": 0, "density": 0.0}
    case.update(kw)
    if not case["shortest"]:
        case["shortest"] = case["longest"]
    if not name:
        del case["name"]
    return case


def listed():
    return [
        # one user, a short conversation: latency and launches count
        _case("decode_1x4k", "decode", batch=1, longest=4000),
        # the benchmark's batch at 32K context
        _case("decode_16x32k", "decode", batch=16, longest=32768),
        # few users with very long documents
        _case("decode_4x256k", "decode", batch=4, longest=262144),
        # a ragged batch of a model without grouped queries, short budget
        _case("decode_mha_32_ragged", "decode", batch=32, kv_heads=32, shortest=4096, longest=131072, budget=2048),
        # a full serving batch over 4-bit pages, streaming heads in their bounded cache
        _case("decode_kv4_64x16k", "decode", batch=64, dtype="bf16", shortest=9001, longest=24011, kv_bits=4, two_way=True),
        # a batch of ordinary short prompts of all lengths
        _case("prefill_ragged_16", "prefill", batch=16, dtype="bf16", shortest=77, longest=3001),
        # one prompt of a few thousand tokens
        _case("prefill_4k", "prefill", longest=4096),
        # the longest prompt of the benchmark
        _case("prefill_64k", "prefill", dtype="bf16", longest=65536),
        # a scheduler that mixes small chunks of a long prompt with decoding
        _case("chunk_512_over_32k", "chunk", dtype="bf16", longest=512, history=32768),
        # large chunks of two users over 8-bit pages, streaming heads in their bounded cache
        _case("chunk_kv8_2x2k", "chunk", batch=2, shortest=1500, longest=2048, history=24001, kv_bits=8, two_way=True),
        # a prompt under a block mask that an outside estimator found
        _case("masked_12k", "masked", dtype="bf16", longest=12345, density=0.3),
        # write-back of a batch of prompts into 4-bit pages
        _case("append_kv4_8", "append", batch=8, shortest=1999, longest=8192, kv_bits=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["decode", "prefill", "chunk", "masked", "append"], [5, 4, 4, 1, 2])[0]
    kw = {"dtype": rng.choice(["fp16", "bf16"])}
    kw["q_heads"], kw["kv_heads"] = rng.choice([(32, 8), (32, 8), (32, 32), (8, 2), (64, 8), (32, 16)])
    if kind == "decode":
        kw["batch"] = _log(rng, 1, 64)
        top = min(262144, (8 << 20) // (kw["batch"] * kw["kv_heads"]))
        kw["longest"] = _log(rng, 1000, max(2000, top))
        kw["shortest"] = rng.choice([0, max(200, kw["longest"] // rng.randint(2, 30))])
        kw["kv_bits"] = rng.choice([16, 16, 8, 4])
        kw["two_way"] = rng.random() < 0.4
        kw["budget"] = 64 * _log(rng, 16, 96)
        if kw["kv_bits"] == 16:
            kw["page"] = rng.choice([64, 64, 64, 32, 128])
    elif kind == "prefill":
        kw["batch"] = _log(rng, 1, 24)
        kw["longest"] = _log(rng, 100, max(200, min(49152, 98304 // kw["batch"])))
        kw["shortest"] = rng.choice([0, max(1, kw["longest"] // rng.randint(2, 40))])
        if kw["q_heads"] == 64:
            kw["longest"] = min(kw["longest"], 32768)
            kw["shortest"] = min(kw["shortest"], 32768)
    elif kind == "chunk":
        kw["batch"] = _log(rng, 1, 8)
        kw["longest"] = _log(rng, 16, 4096)
        kw["shortest"] = rng.choice([0, max(1, kw["longest"] // rng.randint(2, 10))])
        kw["history"] = _log(rng, 300, max(400, min(131072, (1 << 28) // (kw["batch"] * kw["longest"] * kw["q_heads"] // 32))))
        kw["history"] = min(kw["history"], (8 << 20) // (kw["batch"] * kw["kv_heads"]))
        kw["kv_bits"] = rng.choice([16, 16, 8, 4])
        kw["two_way"] = rng.random() < 0.4
    elif kind == "masked":
        kw["batch"] = rng.choice([1, 1, 2, 4])
        kw["longest"] = _log(rng, 500, 24000 // kw["batch"])
        kw["density"] = round(rng.uniform(0.05, 0.8), 3)
    else:
        kw["batch"] = _log(rng, 1, 32)
        kw["longest"] = _log(rng, 1, max(2, min(65536, (1 << 20) // (kw["batch"] * kw["kv_heads"]))))
        kw["shortest"] = rng.choice([0, max(1, kw["longest"] // rng.randint(2, 30))])
        kw["history"] = rng.choice([0, 0, _log(rng, 1, 2000)])
        kw["kv_bits"] = rng.choice([16, 8, 4])
    return _case("", kind, **kw)


# ---- inputs ------------------------------------------------------------------------------------------------------


def _lengths(case):
    """Lengths of the batch: between `shortest` and `longest` (spread over their logarithm, the longest among them)."""
    n, lo, hi = case["batch"], case["shortest"], case["longest"]
    out = [int(round(math.exp(math.log(lo) + ((i * 0.6180339887498949) % 1.0) * (math.log(hi) - math.log(lo)))))
           for i in range(1, n)]
    return [hi] + out


def _dtype(case):
    return torch.float16 if case["dtype"] == "fp16" else torch.bfloat16


def _flags(case):
    half = case["kv_heads"] // 2
    return [1] * half + [0] * (case["kv_heads"] - half)


def _gen(seed, *which):
    x = seed & 0xFFFFFFFF
    for w in which:
        x = (x * 1000003 + w + 12345) & 0x7FFFFFFFFFFF
    g = torch.Generator(device="cuda")
    g.manual_seed(x)
    return g


def _randn(gen, shape, dtype, scale=None):
    out = torch.empty(shape, dtype=dtype, device="cuda")
    rows = max(1, (1 << 26) // max(1, out[0].numel()))
    for r in range(0, shape[0], rows):
        x = torch.randn((min(rows, shape[0] - r),) + tuple(shape[1:]), generator=gen, device="cuda")
        out[r:r + rows] = x if scale is None else x * scale
    return out


def _loudness(case, seed):
    """Factor per (KV head, channel) of the keys: most channels near 1, a few up to 2.5."""
    u = torch.rand((case["kv_heads"], D), generator=_gen(seed, 77), device="cuda")
    return 0.8 + 1.7 * u ** 6


def _kv(case, seed, b, n):
    """K and V of sequence b, [n][Hkv][D]."""
    shape = (n, case["kv_heads"], D)
    g = _gen(seed, 1, b)
    return _randn(g, shape, _dtype(case), _loudness(case, seed)), _randn(g, shape, _dtype(case))


def _q(case, seed, n, which=0):
    return _randn(_gen(seed, 2, which), (n, case["q_heads"], D), _dtype(case))


def _int32(xs):
    return torch.tensor(xs, dtype=torch.int32, device="cuda")


def _cu(lens):
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    return _int32(cu)


def _desc(case):
    return B.AttnDesc(num_q_heads=case["q_heads"], num_kv_heads=case["kv_heads"], streaming_flags=_flags(case),
                      page_size=case["page"], logical_page_size=16, dtype=_dtype(case), sink_tokens=SINK,
                      local_tokens=LOCAL)


def _ring_pages(case):
    return -(-SINK // case["page"]) + -(-LOCAL // case["page"])


def _pools(case, seed, capacity):
    """Empty pools and tables for sequences of up to `capacity[b]` tokens: pages of the shared pool in random order."""
    np_, hkv, bits = case["page"], case["kv_heads"], case["kv_bits"]
    pages = [-(-c // np_) for c in capacity]
    used = sum(pages)
    total = used + max(2, used // 32)
    perm = torch.randperm(total, generator=_gen(seed, 3), device="cuda").to(torch.int32)
    table = torch.zeros((len(pages), max(pages)), dtype=torch.int32, device="cuda")
    at = 0
    for b, p in enumerate(pages):
        table[b, :p] = perm[at:at + p]
        at += p
    n_stream = sum(_flags(case))

    def pool(n, heads):
        if bits == 16:
            return torch.zeros((n, heads, np_, D), dtype=_dtype(case), device="cuda")
        return torch.zeros((n, heads, 64 * D * bits // 8 + 256), dtype=torch.uint8, device="cuda")

    heads = hkv - n_stream if case["two_way"] else hkv
    out = {"k": pool(total, heads), "v": pool(total, heads), "table": table, "ks": None, "vs": None, "ring": None}
    if case["two_way"]:
        ring = _ring_pages(case)
        out["ks"], out["vs"] = pool(len(pages) * ring, n_stream), pool(len(pages) * ring, n_stream)
        out["ring"] = torch.randperm(len(pages) * ring, generator=_gen(seed, 4), device="cuda").to(torch.int32).view(len(pages), ring)
    return out


def _stats_for(case, pools):
    k = pools["k"]
    return torch.zeros((k.shape[0], k.shape[1], case["page"] // 16, 2, D), dtype=_dtype(case), device="cuda")


def _paged(case, pools, stats, seq_lens, b=None):
    table, ring = pools["table"], pools["ring"]
    if b is not None:
        table = table[b:b + 1].clone()
        ring = None if ring is None else ring[b:b + 1].clone()
    heads = pools["k"].shape[1]
    return B.PagedKV(pools["k"], pools["v"], stats, table, seq_lens, pool_heads=0 if heads == case["kv_heads"] else heads,
                     k_pool_stream=pools["ks"], v_pool_stream=pools["vs"], ring_table=ring, kv_bits=case["kv_bits"])


def _write_history(case, desc, pools, stats, b, k, v):
    n = k.shape[0]
    kv = _paged(case, pools, stats, _int32([n]), b)
    B.lserve_append_kv(desc, kv, k, v, _int32([0, n]), _int32([0]), n)


def prepare(case, seed):
    lens = _lengths(case)
    desc = _desc(case)
    kind = case["kind"]
    hq, dt = case["q_heads"], _dtype(case)
    if kind == "decode":
        pools = _pools(case, seed, [n + STEPS for n in lens])
        session = DecodeSession(pools["k"], pools["v"], pools["table"], hq, _flags(case), SINK, LOCAL, case["budget"],
                                logical_page_size=16, reuse_interval=STEPS, k_pool_stream=pools["ks"],
                                v_pool_stream=pools["vs"], ring_table=pools["ring"], kv_bits=case["kv_bits"], dtype=dt)
        new_k, new_v = [], []
        for b, n in enumerate(lens):
            k, v = _kv(case, seed, b, n + STEPS)
            new_k.append(k[n:].clone())
            new_v.append(v[n:].clone())
            _write_history(case, session.desc, pools, session.stats, b, k[:n], v[:n])
        k_new, v_new = torch.stack(new_k, 1).contiguous(), torch.stack(new_v, 1).contiguous()  # [step][batch][Hkv][D]
        return {"case": case, "session": session, "k_new": list(k_new), "v_new": list(v_new),
                "q": [_q(case, seed, case["batch"], i) for i in range(STEPS)],
                "lens": [_int32([n + i for n in lens]) for i in range(STEPS + 1)],
                "cu": _int32(list(range(case["batch"] + 1))),
                "out": [torch.empty((case["batch"], hq, D), dtype=dt, device="cuda") for _ in range(STEPS)]}
    if kind in ("prefill", "masked"):
        ks, vs = zip(*[_kv(case, seed, b, n) for b, n in enumerate(lens)])
        q = _q(case, seed, sum(lens))
        state = {"case": case, "desc": desc, "q": q, "k": torch.cat(ks), "v": torch.cat(vs), "cu": _cu(lens),
                 "longest": max(lens), "out": torch.empty_like(q)}
        if kind == "masked":
            state["mask"] = _block_mask(case, seed)
            need = B.lserve_masked_prefill_workspace_bytes(desc, len(lens), sum(lens), max(lens), 2, state["mask"].nnz)
            state["ws"] = torch.empty((max(16, need),), dtype=torch.uint8, device="cuda")
        return state
    if kind == "chunk":
        hist = case["history"]
        pools = _pools(case, seed, [hist + n for n in lens])
        stats = _stats_for(case, pools)
        new_k, new_v = [], []
        for b, n in enumerate(lens):
            k, v = _kv(case, seed, b, hist + n)
            new_k.append(k[hist:].clone())
            new_v.append(v[hist:].clone())
            _write_history(case, desc, pools, stats, b, k[:hist], v[:hist])
        q = _q(case, seed, sum(lens))
        return {"case": case, "desc": desc, "kv": _paged(case, pools, stats, _int32([hist] * len(lens))), "q": q,
                "k": torch.cat(new_k), "v": torch.cat(new_v), "cu": _cu(lens), "longest": max(lens),
                "out": torch.empty_like(q)}
    assert kind == "append"
    hist = case["history"]
    pools = _pools(case, seed, [hist + n for n in lens])
    stats = _stats_for(case, pools)
    new_k, new_v = [], []
    for b, n in enumerate(lens):
        k, v = _kv(case, seed, b, hist + n)
        new_k.append(k[hist:].clone())
        new_v.append(v[hist:].clone())
        if hist:
            _write_history(case, desc, pools, stats, b, k[:hist], v[:hist])
    return {"case": case, "desc": desc, "kv": _paged(case, pools, stats, _int32([hist + n for n in lens])),
            "k": torch.cat(new_k), "v": torch.cat(new_v), "cu": _cu(lens), "start": _int32([hist] * len(lens)),
            "longest": max(lens)}


def _mask_tiles(case, seed, b, n):
    """Kept key tiles of the two masks of sequence b: [2][tiles][tiles] bool, first tile, a band of four and `density`
    of the rest."""
    tiles = -(-n // TILE)
    rnd = torch.rand((2, tiles, tiles), generator=_gen(seed, 5, b), device="cuda") < case["density"]
    i = torch.arange(tiles, device="cuda")
    keep = rnd | (i[None, :] == 0) | (i[:, None] - i[None, :] < 4)
    return keep & (i[None, :] <= i[:, None])


def _block_mask(case, seed):
    lens = _lengths(case)
    rows, starts, counts, cols = 0, [0], [], []
    per_seq = [_mask_tiles(case, seed, b, n) for b, n in enumerate(lens)]
    for keep in per_seq:
        rows += keep.shape[1]
        starts.append(rows)
    for m in range(2):
        for keep in per_seq:
            counts.append(keep[m].sum(1))
            cols.append(keep[m].nonzero()[:, 1])
    row_ptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cat(counts).cumsum(0)]).to(torch.int32)
    return B.BlockMask(_int32(_head_mask(case)), _int32(starts), row_ptr, torch.cat(cols).to(torch.int32).contiguous(), 2, rows)


def _head_mask(case):
    """Query heads of dense KV heads take the two listed masks in turn; streaming heads keep their own pattern."""
    n = case["q_heads"] // case["kv_heads"]
    flags = _flags(case)
    return [-1 if flags[h // n] else h % 2 for h in range(case["q_heads"])]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "decode":
        s = state["session"]
        s.restart()
        for i in range(STEPS):
            s.append(state["k_new"][i], state["v_new"][i], state["cu"], state["lens"][i], 1)
            s.out = state["out"][i]
            s.step(state["q"][i], state["lens"][i + 1], state["lens"][i])
        return {"out": state["out"], "pages": s.sel_pages}
    if kind == "prefill":
        B.lserve_sparse_prefill(state["desc"], state["q"], state["k"], state["v"], state["cu"], state["longest"], state["out"])
        return state["out"]
    if kind == "masked":
        B.lserve_sparse_prefill_masked(state["desc"], state["mask"], state["q"], state["k"], state["v"], state["cu"],
                                       state["longest"], state["out"], None, state["ws"])
        return state["out"]
    if kind == "chunk":
        B.lserve_sparse_prefill_chunk(state["desc"], state["kv"], state["q"], state["k"], state["v"], state["cu"],
                                      state["longest"], state["out"])
        return state["out"]
    kv = state["kv"]
    B.lserve_append_kv(state["desc"], kv, state["k"], state["v"], state["cu"], state["start"], state["longest"])
    return {"k": kv.k_pool, "v": kv.v_pool, "stats": kv.stats}


# ---- floors --------------------------------------------------------------------------------------------------------


def _row_bytes(case):
    """Bytes of one stored token row of one head, scale and zero point included."""
    return 2 * D if case["kv_bits"] == 16 else D * case["kv_bits"] // 8 + 4


def _streaming_pairs(first, n):
    """(query, key) pairs a streaming head attends for the queries at positions first .. first + n - 1."""
    s, w = SINK // TILE, LOCAL // TILE
    total, t = 0, first
    while t < first + n:
        tile = t // TILE
        end = min(first + n, (tile + 1) * TILE)
        band = max(0, tile - w + 1)
        whole = min(s, band) + tile - band  # tiles below the diagonal one
        total += sum(whole * TILE + u - tile * TILE + 1 for u in range(t, end))
        t = end
    return total


def work(case):
    """Per decode step the listed pages are read again: between two steps of a layer lie all the others."""
    lens = _lengths(case)
    hq, hkv = case["q_heads"], case["kv_heads"]
    n_stream = sum(_flags(case))
    group, row = hq // hkv, _row_bytes(case)
    if case["kind"] == "decode":
        np_, k_pages = case["page"], case["budget"] // case["page"]
        s, w = -(-SINK // np_), -(-LOCAL // np_)
        tokens = stats = 0
        for n in lens:
            stats += -(-(n + 1) // 16) * (hkv - n_stream) * 2 * D * 2
            for i in range(1, STEPS + 1):
                length = n + i
                pages = -(-length // np_)
                tail = length - (pages - 1) * np_
                sel = min(pages, k_pages + pages - -(-(n + 1) // np_))
                tokens += (hkv - n_stream) * ((sel - 1) * np_ + tail)
                tokens += n_stream * ((min(pages, s + w) - 1) * np_ + tail)
        io = STEPS * case["batch"] * (2 * hq * D * 2 + 2 * hkv * (2 * D + row))
        return {"bytes": 2 * row * tokens + stats + io,
                "flops": 4 * D * group * tokens + (stats // 2) * 2 * group}
    total = sum(lens)
    if case["kind"] == "append":
        logical = sum(-(-(case["history"] + n) // 16) - case["history"] // 16 for n in lens)
        return {"bytes": 2 * total * hkv * (2 * D + row) + logical * (hkv - n_stream) * 2 * D * 2, "flops": 0}
    hist = case["history"] if case["kind"] == "chunk" else 0
    dense = sum(n * hist + n * (n + 1) // 2 for n in lens)
    if case["kind"] == "masked":
        dense = 0
        for n in lens:
            tiles = -(-n // TILE)
            kept = sum(min(i, 3) + (1 + (i - 4) * case["density"] if i > 3 else 0) for i in range(tiles))
            dense += int(kept * TILE * TILE + n * (TILE + 1) // 2)
    stream = sum(_streaming_pairs(hist, n) for n in lens)
    hist_rows = hist * (hkv - n_stream) + min(hist, SINK + LOCAL) * n_stream
    return {"bytes": 2 * total * (hq + hkv) * D * 2 + case["batch"] * 2 * hist_rows * row,
            "flops": 4 * D * group * (dense * (hkv - n_stream) + stream * n_stream)}


def tolerance(case):
    """What the 16-bit types leave open, about four times the error against `exact`: a decode step only rounds its
    output to them (2.1e-4 in fp16, 1.7e-3 in bf16; over quantised pages also the softmax weights, to fp16: 4.9e-4),
    prefill its softmax weights and scaled queries too (4.6e-4 and 2.8e-3).  A selected page may differ where two scores
    tie in fp32.  A write-back moves, rounds and compares whole values: the same bytes."""
    if case["kind"] == "append":
        return "exact"
    fp16 = case["dtype"] == "fp16"
    if case["kind"] == "decode":
        return {"rel": (1e-3 if case["kv_bits"] == 16 else 2e-3) if fp16 else 7e-3, "differ": 2e-3}
    return {"rel": 2e-3 if fp16 else 1.1e-2}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------


def _as_stored(case, x):
    """Rows as the cache keeps them: 16-bit rows as they are, quantised rows as code * scale + zero, in 64 bits."""
    x = x.double()
    if case["kv_bits"] == 16:
        return x
    top = float(2 ** case["kv_bits"] - 1)
    big = 65504.0
    zero = x.amin(-1, keepdim=True).clamp(-big, big).half().double()
    span = (x.amax(-1, keepdim=True) - zero).float().double()
    scale = (span / top).float().clamp(max=big).half().double()
    code = ((x - zero).float().double() / scale.clamp(min=1e-30)).float().double().round().clamp(0, top)
    return torch.where(scale > 0, code, torch.zeros_like(code)) * scale + zero


def _attend(q, k, v, allowed):
    """softmax(q k^T / sqrt(D)) v for [n][D], [m][D], [m][D] under a boolean [n][m] mask."""
    s = (q @ k.T) / math.sqrt(D)
    s = s.masked_fill(~allowed, -math.inf)
    p = torch.exp(s - s.amax(-1, keepdim=True))
    return (p @ v) / p.sum(-1, keepdim=True)


def _exact_prefill(case, seed):
    lens = _lengths(case)
    hist = case["history"] if case["kind"] == "chunk" else 0
    hq, hkv, flags = case["q_heads"], case["kv_heads"], _flags(case)
    group = hq // hkv
    q_all = _q(case, seed, sum(lens))
    out = torch.empty((sum(lens), hq, D), dtype=torch.float64, device="cuda")
    head_mask = _head_mask(case) if case["kind"] == "masked" else [-1] * hq
    s, w = SINK // TILE, LOCAL // TILE
    row = 0
    for b, n in enumerate(lens):
        k, v = _kv(case, seed, b, hist + n)
        keep = _mask_tiles(case, seed, b, n) if case["kind"] == "masked" else None
        for hk in range(hkv):
            kd, vd = k[:, hk].double(), v[:, hk].double()
            if hist:
                kd[:hist], vd[:hist] = _as_stored(case, k[:hist, hk]), _as_stored(case, v[:hist, hk])
            for h in range(hk * group, (hk + 1) * group):
                qd = q_all[row:row + n, h].double()
                for r in range(0, n, 1024):
                    t = torch.arange(hist + r, hist + min(n, r + 1024), device="cuda")
                    end = hist + min(n, r + 1024)
                    u = torch.arange(end, device="cuda")
                    allowed = u[None, :] <= t[:, None]
                    if head_mask[h] >= 0:
                        allowed &= keep[head_mask[h]][t[:, None] // TILE, u[None, :] // TILE]
                    elif flags[hk]:
                        allowed &= (u[None, :] // TILE < s) | (u[None, :] // TILE > t[:, None] // TILE - w)
                    out[row + r:row + r + len(t), h] = _attend(qd[r:r + 1024], kd[:end], vd[:end], allowed)
        row += n
    return out


def _exact_decode(case, seed):
    lens = _lengths(case)
    hq, hkv, flags, np_ = case["q_heads"], case["kv_heads"], _flags(case), case["page"]
    group, K = hq // hkv, case["budget"] // np_
    s, w = -(-SINK // np_), -(-LOCAL // np_)
    q = [_q(case, seed, case["batch"], i).double() for i in range(STEPS)]
    out = [torch.empty((case["batch"], hq, D), dtype=torch.float64, device="cuda") for _ in range(STEPS)]
    pages = torch.full((case["batch"], hkv, K), -1, dtype=torch.int32, device="cuda")
    for b, n in enumerate(lens):
        k, v = _kv(case, seed, b, n + STEPS)
        first = n + 1  # length at the selector run
        P0 = -(-first // np_)
        for hk in range(hkv):
            if flags[hk]:
                chosen = None
            elif P0 <= K:
                chosen = torch.arange(P0, device="cuda")
            else:
                rows = torch.full((P0 * np_, D), math.nan, dtype=torch.float64, device="cuda")
                rows[:first] = k[:first, hk].double()
                logical = rows.view(-1, 16, D)
                live = ~logical.isnan()
                top = torch.where(live, logical, torch.full_like(logical, -math.inf)).amax(1)
                low = torch.where(live, logical, torch.full_like(logical, math.inf)).amin(1)
                used = -(-first // 16)
                qg = q[0][b, hk * group:(hk + 1) * group]
                sc = torch.full((P0 * np_ // 16,), -math.inf, dtype=torch.float64, device="cuda")
                sc[:used] = (top[:used] @ qg.clamp(min=0).T + low[:used] @ qg.clamp(max=0).T).amax(1)
                sc = sc.view(P0, -1).amax(1)[:P0 - 1]
                best = torch.sort(sc, descending=True, stable=True).indices[:K - 1]
                chosen = torch.cat([best.sort().values, torch.tensor([P0 - 1], device="cuda")])
            if chosen is not None:
                pages[b, hk, :len(chosen)] = chosen.to(torch.int32)
            for i in range(STEPS):
                length = n + 1 + i
                P = -(-length // np_)
                if chosen is None:
                    head = min(s, P)
                    listed_pages = torch.cat([torch.arange(head, device="cuda"),
                                              torch.arange(max(head, P - w), P, device="cuda")])
                else:
                    listed_pages = torch.cat([chosen, torch.arange(P0, P, device="cuda")])
                tok = (listed_pages[:, None] * np_ + torch.arange(np_, device="cuda")).flatten()
                tok = tok[tok < length]
                kd, vd = _as_stored(case, k[tok, hk]), _as_stored(case, v[tok, hk])
                h = slice(hk * group, (hk + 1) * group)
                sc = (q[i][b, h] @ kd.T) / math.sqrt(D)
                p = torch.exp(sc - sc.amax(-1, keepdim=True))
                out[i][b, h] = (p @ vd) / p.sum(-1, keepdim=True)
    return {"out": out, "pages": pages}


def exact(case, seed):
    if case["kind"] == "append":
        return None  # bytes and whole values, compared bit for bit
    if case["kind"] == "decode":
        # a few small products per (sequence, head, step): some thousands are quick
        return _exact_decode(case, seed) if case["batch"] * case["kv_heads"] <= 1100 else None
    if work(case)["flops"] > 2.5e13:
        return None
    return _exact_prefill(case, seed)
