"""A selector run whose budget covers the page table is one launch: the lists and the statistics of the general route, which a
wider table takes."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("page,logical", [(64, 16), (16, 16), (32, 4), (128, 16)])
@pytest.mark.parametrize("two_way", [False, True])
def test_budget_covers_the_table(dtype, page, logical, two_way):
    import paper_2502_14866_amd as L

    L.load_library()
    dev, hkv, group = torch.device("cuda:0"), 3, 2
    flags, pages = [0, 1, 0], 17
    lens = [1, logical, logical + 1, page, page + 1, pages * page - 1, pages * page, 5 * page + 3, 9]
    valid = [0, logical - 1, logical, page, 0, pages * page - 5, 3 * logical + 1, 5 * page + 3, 12]  # some ahead of the length
    B = len(lens)
    g = torch.Generator().manual_seed(page + logical)
    heads = 2 if two_way else hkv
    k = torch.randn((B * pages, heads, page, 128), generator=g).to(dtype).to(dev)
    table = torch.randperm(B * pages, generator=g).to(torch.int32).reshape(B, pages).to(dev)
    q = torch.randn((B, group * hkv, 128), generator=g).to(dtype).to(dev)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    desc = L.AttnDesc(group * hkv, hkv, flags, page_size=page, logical_page_size=logical, dtype=dtype, sink_tokens=page,
                      local_tokens=2 * page)
    side = torch.zeros((B * 3, 1, page, 128), dtype=dtype, device=dev) if two_way else None
    ring = torch.arange(B * 3, dtype=torch.int32, device=dev).reshape(B, 3) if two_way else None
    K = pages + 2
    got = []
    for width, stale in ((pages, True), (4 * pages, True), (pages, False), (4 * pages, False)):
        wide = torch.cat([table, torch.zeros((B, width - pages), dtype=torch.int32, device=dev)], 1).contiguous()
        stats = torch.full((B * pages, heads, page // logical, 2, 128), 7.0, dtype=dtype, device=dev)
        kv = L.PagedKV(k, k, stats, wide, i32(lens), pool_heads=2 if two_way else 0, k_pool_stream=side, v_pool_stream=side,
                       ring_table=ring)
        sel = torch.full((B, hkv, K), -7, dtype=torch.int32, device=dev)
        cnt, at = torch.full((B, hkv), -7, dtype=torch.int32, device=dev), torch.full((B,), -7, dtype=torch.int32, device=dev)
        ws = torch.empty((max(16, L.lserve_workspace_bytes(L.LSERVE_CALL_SELECT_PAGES, desc, B, width, K, 0)),), dtype=torch.uint8, device=dev)
        L.lserve_select_pages(desc, kv, q, K * page, sel, cnt, at, None, ws, stats_valid_len=i32(valid) if stale else None)
        torch.cuda.synchronize()
        got.append((sel, cnt, at, stats))
    for a, b in ((0, 1), (2, 3)):
        for x, y in zip(got[a], got[b]):
            assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
    assert not torch.equal(got[0][3], got[2][3])  # some were out of date


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("batch,pages", [(100, 33), (683, 9)])
def test_more_work_than_workgroups_to_share_it_out(dtype, batch, pages):
    """So many lists that a workgroup takes several turns over the logical pages of its own, of which all, some or none are out of date."""
    import paper_2502_14866_amd as L

    L.load_library()
    dev, hkv = torch.device("cuda:0"), 3
    g = torch.Generator().manual_seed(batch)
    lens = torch.randint(1, pages * 64 + 1, (batch,), generator=g).to(torch.int32)
    lens[0] = pages * 64
    valid = (lens * torch.rand(batch, generator=g) * (torch.arange(batch) % 3)).to(torch.int32).to(dev)
    table = torch.randperm(batch * pages, generator=g).to(torch.int32).reshape(batch, pages).to(dev)
    k = torch.randn((batch * pages, hkv, 64, 128), generator=torch.Generator(device=dev).manual_seed(1), device=dev, dtype=dtype)
    q = torch.zeros((batch, 2 * hkv, 128), dtype=dtype, device=dev)
    desc = L.AttnDesc(2 * hkv, hkv, [0, 1, 0], dtype=dtype)
    got = []
    for width in (pages, 4 * pages):
        wide = torch.cat([table, torch.zeros((batch, width - pages), dtype=torch.int32, device=dev)], 1).contiguous()
        stats = torch.full((batch * pages, hkv, 4, 2, 128), 7.0, dtype=dtype, device=dev)
        kv = L.PagedKV(k, k, stats, wide, lens.to(dev))
        sel = torch.full((batch, hkv, pages), -7, dtype=torch.int32, device=dev)
        cnt, at = torch.full((batch, hkv), -7, dtype=torch.int32, device=dev), torch.full((batch,), -7, dtype=torch.int32, device=dev)
        ws = torch.empty((L.lserve_workspace_bytes(L.LSERVE_CALL_SELECT_PAGES, desc, batch, width, pages, 0),), dtype=torch.uint8, device=dev)
        L.lserve_select_pages(desc, kv, q, pages * 64, sel, cnt, at, None, ws, stats_valid_len=valid)
        torch.cuda.synchronize()
        got.append((sel, cnt, at, stats))
    for x, y in zip(*got):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
    assert (got[0][3] != 7.0).any()
