"""Chunks of many rows over quantised pages, whose history is turned into 16-bit pages first (scratch of
lserve_sparse_prefill_chunk_scratch): sampled rows against the oracle."""
import pytest

import test_gpu_paged_shapes as paged

pytestmark = pytest.mark.gpu

CASES = [  # heads, KV heads, history, new tokens
    (32, 8, (1600,), (700,)),                     # whole pages of history
    (32, 8, (2501, 1999), (900, 801)),            # off the pages
    (8, 8, (1501, 0, 3), (2300, 2100, 2049)),     # no groups; no history, less than a page of it
    (12, 4, (1700, 2000, 64), (1500, 0, 2000)),   # an idle sequence; sink and local pages are all there is
    (64, 8, (2047,), (400,)),
    (8, 1, (3001,), (300,)),                      # no streaming head
    (32, 8, (4400, 4100), (2500, 2600)),          # whole workgroups in one slice over the 16-bit pages
    # dense walks over the 16-bit pages cut into pieces, streaming heads in the launch that puts them together
    (32, 8, (16001,), (512,)),
    (8, 2, (30000,), (1500,)),
    (12, 4, (30001,), (900,)),                    # groups of three
    (16, 4, (20001, 3000), (900, 300)),           # sequences of different lengths
]
PIECES = (5, 7, 8, 9, 10)


def _scratch(desc, heads, hkv, hist, fresh, bits, sink, local):
    """The plan, and the scratch it takes: expanded pages, ring and tables, then the pieces."""
    import paper_2502_14866_amd as L

    pages = max(-(-(h + n) // 64) for h, n in zip(hist, fresh))
    plan = L.lserve_probe_prefill_plan(desc, len(hist), sum(fresh), max(fresh), pages, bits)
    streaming, ring = hkv // 2, sink // 64 + local // 64
    whole = lambda x: -(-x // 256) * 256
    slab, b, group = 64 * 128 * 2, len(hist), heads // hkv
    per_block = 4 if group % 4 == 0 else 2 if group % 2 == 0 else 1
    expanded = (2 * whole(b * pages * (hkv - streaming) * slab) + 2 * whole(b * ring * streaming * slab) + whole(4 * b * pages)
                + whole(4 * b * ring))
    return plan, expanded, plan["pieces"] * (hkv - streaming) * (group // per_block) * 8 * (32 * 128 + 64) * 4


@pytest.mark.parametrize("dtype,bits", [("fp16", 8), ("bf16", 8), ("fp16", 4), ("bf16", 4)])
@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_chunks_over_expanded_pages(case, dtype, bits, two_way, monkeypatch):
    import paper_2502_14866_amd as L
    import paper_2502_14866_amd.binding as B

    heads, hkv, hist, fresh = CASES[case]
    if hkv == 1 and two_way:
        pytest.skip("a bounded pool is for streaming heads")
    used = []
    take = B._chunk_scratch

    def recorded(*args):
        used.append(take(*args))
        if used[-1] is not None:
            used[-1].fill_(0xff)  # of any contents
        return used[-1]
    monkeypatch.setattr(B, "_chunk_scratch", recorded)
    monkeypatch.setattr(paged, "CASES", [(heads, hkv, hist, fresh, {8: None, 4: None})])
    paged.test_chunks_in_every_launch_shape(0, dtype, bits, two_way)
    desc = L.AttnDesc(heads, hkv, [1 if h < hkv // 2 else 0 for h in range(hkv)], sink_tokens=paged.SINK, local_tokens=paged.LOCAL)
    plan, expanded, pieces = _scratch(desc, heads, hkv, hist, fresh, bits, paged.SINK, paged.LOCAL)
    assert plan["expand"] and bool(plan["pieces"]) == (case in PIECES) and plan["apart"] == (case in PIECES and hkv > 1)
    assert len(used) == 1 and used[0].numel() == expanded + pieces


@pytest.mark.parametrize("two_way", [False, True])
def test_sequences_without_new_tokens_are_not_expanded(two_way, monkeypatch):
    import paper_2502_14866_amd.binding as B

    heads, hkv, hist, fresh = CASES[3]
    idle = fresh.index(0)
    used, take = [], B._chunk_scratch
    monkeypatch.setattr(B, "_chunk_scratch", lambda *args: used.append(take(*args).fill_(0xff)) or used[-1])
    monkeypatch.setattr(paged, "CASES", [(heads, hkv, hist, fresh, {8: None, 4: None})])
    paged.test_chunks_in_every_launch_shape(0, "fp16", 8, two_way)
    pages = max(-(-(h + n) // 64) for h, n in zip(hist, fresh))
    per_seq = pages * (hkv - hkv // 2) * 64 * 128 * 2
    k = used[0][:len(hist) * per_seq].reshape(len(hist), per_seq).cpu()
    assert (k[idle] == 0xff).all() and all((k[b] != 0xff).any() for b in range(len(hist)) if b != idle)
