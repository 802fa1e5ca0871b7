"""Chunks over histories long enough that their dense walks are cut into pieces (lserve_sparse_prefill_chunk_scratch): every form
of cache, groups of heads that fill a workgroup or not, batches whose sequences differ in everything, sampled rows against the
oracle, and the call without scratch beside it, whose streaming heads have the same bits."""
import pytest
import torch

import test_gpu_paged_shapes as paged

pytestmark = pytest.mark.gpu

CASES = [  # heads, KV heads, history, new tokens
    (32, 8, (12000,), (1,)),                                 # one row
    (32, 8, (12096,), (64,)),                                # whole tiles
    (32, 8, (14100, 14100), (190, 190)),                     # alike, off the tiles
    (8, 8, (12000,), (300,)),                                # no groups: a block is four tiles
    (12, 2, (13500, 70), (130, 65)),                         # six heads per group: two of them and two tiles to a block
    (12, 4, (0, 26000, 3, 700), (200, 17, 0, 64)),           # idle and empty sequences beside a long one
    (64, 8, (14900,), (77,)),                                # eight heads per group: two workgroups to a block
    # two sequences to some lanes, most of them idle (16-bit pages stay with whole walks)
    (4, 2, tuple(977 * i % 600 + 40000 * int(i == 46) for i in range(66)), tuple(3 * int(i % 23 == 0) for i in range(66))),
]


@pytest.mark.parametrize("dtype,bits,two_way", [("fp16", 16, False), ("bf16", 16, True), ("bf16", 8, False), ("fp16", 4, True)])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_chunks_in_pieces(case, dtype, bits, two_way, monkeypatch):
    import paper_2502_14866_amd as L
    import paper_2502_14866_amd.binding as B

    heads, hkv, hist, fresh = CASES[case]
    used = []
    take = B._chunk_scratch

    def recorded(*args):
        used.append(take(*args))
        if used[-1] is not None:
            used[-1].fill_(0xff)  # of any contents
        return used[-1]
    monkeypatch.setattr(B, "_chunk_scratch", recorded)
    monkeypatch.setattr(paged, "CASES", [(heads, hkv, hist, fresh, {16: None, 8: None, 4: None})])
    paged.test_chunks_in_every_launch_shape(0, dtype, bits, two_way)
    desc = L.AttnDesc(heads, hkv, [1 if h < hkv // 2 else 0 for h in range(hkv)], sink_tokens=paged.SINK, local_tokens=paged.LOCAL)
    pages = max(-(-(h + n) // 64) for h, n in zip(hist, fresh))
    plan = L.lserve_probe_prefill_plan(desc, len(hist), sum(fresh), max(fresh), pages, bits)
    assert len(used) == 1 and not plan["expand"]
    if bits == 16 and len(hist) > 64:
        assert used[0] is None and not plan["pieces"]
    else:
        group = heads // hkv
        per_block = 4 if group % 4 == 0 else 2 if group % 2 == 0 else 1
        assert plan["pieces"] and plan["apart"]
        assert used[0].numel() == plan["pieces"] * (hkv - hkv // 2) * (group // per_block) * 8 * (32 * 128 + 64) * 4


def test_paged_prefill_in_pieces_repeats_itself_and_agrees_with_whole_walks():
    """Five times on the same data with scratch: the same bits; without (an empty one): the same but for rounding."""
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(7)
    n, new = 20000, 100
    rnd = lambda *s: torch.randn(s, generator=g, device=dev).to(torch.float16)
    k, v, q = rnd(313, 8, 64, 128), rnd(313, 8, 64, 128), rnd(new, 32, 128)
    desc = L.AttnDesc(32, 8, [1, 1, 1, 1, 0, 0, 0, 0])
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    kv = L.PagedKV(k, v, None, torch.randperm(313, generator=g, device=dev).to(torch.int32).reshape(1, -1), i32([n]))
    outs = []
    for i in range(6):
        out, lse = torch.full_like(q, float("nan")), torch.full((32, new), float("nan"), device=dev)
        L.lserve_sparse_prefill_paged(desc, kv, q, i32([0, new]), new, n, out, lse,
                                      scratch=torch.empty((0,), dtype=torch.uint8, device=dev) if i == 5 else None)
        outs.append((out, lse))
    torch.cuda.synchronize()
    for out, lse in outs[1:5]:
        assert torch.equal(out, outs[0][0]) and torch.equal(lse, outs[0][1])
    # streaming heads keep the slices of the launch without scratch
    assert torch.equal(outs[5][0][:, :16], outs[0][0][:, :16]) and torch.equal(outs[5][1][:16], outs[0][1][:16])
    assert not torch.equal(outs[5][1][16:], outs[0][1][16:])
    # weights and outputs are rounded to fp16 on both sides: 2^-11 of the largest output twice
    assert (outs[5][0].float() - outs[0][0].float()).abs().max() <= 2 ** -10 * outs[0][0].float().abs().max()
    assert (outs[5][1] - outs[0][1]).abs().max() <= 1e-5 * outs[0][1].abs().max()


def test_the_workspace_of_paged_prefill_is_not_used():
    """Callers may hand one to calls on several streams: however large, it is left as it is."""
    import ctypes

    import paper_2502_14866_amd as L
    from paper_2502_14866_amd.binding import lserve_chunk_scratch_bytes

    lib = L.load_library()
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(9)
    n, new = 20000, 100
    rnd = lambda *s: torch.randn(s, generator=g, device=dev).to(torch.float16)
    k, v, q = rnd(313, 8, 64, 128), rnd(313, 8, 64, 128), rnd(new, 32, 128)
    desc = L.AttnDesc(32, 8, [1, 1, 1, 1, 0, 0, 0, 0])
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    kv, cu = L.PagedKV(k, v, None, torch.arange(313, device=dev).to(torch.int32).reshape(1, -1), i32([n])), i32([0, new])
    need = lserve_chunk_scratch_bytes(desc, 1, new, new, 313)
    assert need > 0
    ws = torch.full((2 * need,), 0x5a, dtype=torch.uint8, device=dev)
    outs = [torch.empty_like(q) for _ in range(4)]
    L.lserve_sparse_prefill_paged(desc, kv, q, cu, new, n, outs[0], None, ws)
    L.lserve_sparse_prefill_paged(desc, kv, q, cu, new, n, outs[1])
    stream = torch.cuda.current_stream().cuda_stream
    for out, size in ((outs[2], ws.numel()), (outs[3], 0)):  # the entry point in C
        assert lib.lserve_sparse_prefill_paged(desc.c(), kv.c(), q.data_ptr(), cu.data_ptr(), new, new, n, out.data_ptr(), None,
                                               ws.data_ptr() if size else None, ctypes.c_size_t(size), stream) == 0
    torch.cuda.synchronize()
    assert (ws == 0x5a).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[2], outs[3])
