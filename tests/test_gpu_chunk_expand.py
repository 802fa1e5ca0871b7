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
]


@pytest.mark.parametrize("dtype,bits", [("fp16", 8), ("bf16", 8), ("fp16", 4), ("bf16", 4)])
@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_chunks_over_expanded_pages(case, dtype, bits, two_way, monkeypatch):
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
    pages = max(-(-(h + n) // 64) for h, n in zip(hist, fresh))
    dense = hkv - hkv // 2
    assert used[0] is not None and used[0].numel() >= len(hist) * pages * dense * 2 * 64 * 128 * 2


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
