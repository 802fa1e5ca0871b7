"""Decode over 16-bit pages for every group size, scores from matrix products or from the vector pipe: lengths at the edges of a
wavefront's tokens, slots past the end that hold not-a-numbers, maxima that move with every page, a query head that is not a number."""
import numpy as np
import pytest
import torch

from parity import assert_attention_close, assert_lse_close

pytestmark = pytest.mark.gpu

LENGTHS = (1, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 127, 128, 129, 300, 511)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("page", [32, 64, 128])
@pytest.mark.parametrize("group", [1, 2, 3, 4, 5, 6, 7, 8])
def test_every_group_size_at_the_edges_of_a_page(group, page, dtype):
    import paper_2502_14866_amd as L

    L.load_library()
    dev, hkv, B = torch.device("cuda:0"), 2, len(LENGTHS)
    heads = group * hkv
    pages = -(-max(LENGTHS) // page)
    g = torch.Generator().manual_seed(17 * group + page)
    table = torch.randperm(B * pages, generator=g).to(torch.int32).reshape(B, pages)
    k = torch.full((B * pages, hkv, page, 128), float("nan"), dtype=dtype)
    v = torch.full((B * pages, hkv, page, 128), float("nan"), dtype=dtype)
    q = torch.randn((B, heads, 128), generator=g).to(dtype)
    q[2, heads - 1] = float("nan")
    ref, lse = np.zeros((B, heads, 128)), np.zeros((B, heads))
    for b, n in enumerate(LENGTHS):
        kb, vb = torch.randn((n, hkv, 128), generator=g), torch.randn((n, hkv, 128), generator=g).to(dtype)
        kb = (kb * (0.2 + torch.arange(n) / 64)[:, None, None]).to(dtype)  # the largest score lies in the last pages
        pos = torch.arange(n)
        at = table[b].long()[pos // page]
        k[at, :, pos % page], v[at, :, pos % page] = kb, vb
        for h in range(heads):
            s = kb[:, h // group].double() @ q[b, h].double() / np.sqrt(128)
            ref[b, h] = (torch.softmax(s, 0) @ vb[:, h // group].double()).numpy()
            lse[b, h] = torch.logsumexp(s, 0).item()
    # every page is a local one: no selection
    desc = L.AttnDesc(heads, hkv, [1] * hkv, page_size=page, logical_page_size=16, dtype=dtype, sink_tokens=page,
                      local_tokens=pages * page)
    kv = L.PagedKV(k.to(dev), v.to(dev), None, table.to(dev), torch.tensor(LENGTHS, dtype=torch.int32, device=dev))
    out = torch.empty((B, heads, 128), dtype=dtype, device=dev)
    out_lse = torch.empty((B, heads), dtype=torch.float32, device=dev)
    ws = torch.zeros((max(16, L.lserve_workspace_bytes(L.LSERVE_CALL_SPARSE_DECODE, desc, B, pages, 1, 0)),), dtype=torch.uint8, device=dev)
    L.lserve_sparse_decode(desc, kv, q.to(dev), None, None, None, out, out_lse, ws)
    torch.cuda.synchronize()
    assert torch.isnan(out[2, heads - 1]).all()
    out[2, heads - 1], ref[2, heads - 1], out_lse[2, heads - 1], lse[2, heads - 1] = 0, 0, 0, 0
    assert_attention_close(out, ref, f"group {group} page {page}")
    assert_lse_close(out_lse, lse, f"group {group} page {page} lse")
