"""The binding's native calls: what they refuse is refused as by the calls through ctypes, before anything is launched."""
import pytest
import torch

import paper_2502_14866_amd as L
from paper_2502_14866_amd import binding as B


def _problem():
    k = torch.zeros((8, 2, 64, 128), dtype=torch.float16)
    kv = L.PagedKV(k, k.clone(), torch.zeros((8, 2, 4, 2, 128), dtype=torch.float16), torch.zeros((2, 4), dtype=torch.int32),
                   torch.ones((4,), dtype=torch.int32)[:2])
    i32 = lambda *s: torch.zeros(s, dtype=torch.int32)
    a = {"desc": L.AttnDesc(4, 2, [1, 0]), "kv": kv, "q": torch.zeros((2, 4, 128), dtype=torch.float16), "sel": i32(2, 2, 4),
         "cnt": i32(2, 2), "ssl": i32(4), "ws": torch.zeros((16,), dtype=torch.uint8), "new": torch.zeros((2, 2, 128), dtype=torch.float16),
         "cu": i32(4)}
    calls = {
        "append": lambda **k: (lambda a: L.lserve_append_kv(a["desc"], a["kv"], a["new"], a["new"], a["cu"], a["ssl"], 0, 0))({**a, **k}),
        "select": lambda **k: (lambda a: L.lserve_select_pages(a["desc"], a["kv"], a["q"], 256, a["sel"], a["cnt"], a["ssl"], None, a["ws"], 0))({**a, **k}),
        "decode": lambda **k: (lambda a: L.lserve_sparse_decode(a["desc"], a["kv"], a["q"], a["sel"], a["cnt"], a["ssl"], torch.zeros_like(a["q"]), None, a["ws"], 0))({**a, **k}),
    }
    return a, calls


@pytest.mark.parametrize("call,code", [("append", -1), ("select", -3), ("decode", -3)])
def test_library_errors_come_back(call, code):
    _, calls = _problem()  # a launch bound of 0, workspaces too small
    with pytest.raises(B.LserveError) as e:
        calls[call]()
    assert e.value.code == code


@pytest.mark.parametrize("call", ["append", "select", "decode"])
def test_objects_that_are_no_contiguous_tensors(call):
    a, calls = _problem()
    other = {"append": "new"}.get(call, "q")
    with pytest.raises(ValueError):
        calls[call](**{other: torch.zeros((2, 128, 4), dtype=torch.float16).transpose(1, 2)})
    with pytest.raises(TypeError):
        calls[call](**{other: [1, 2, 3]})
    with pytest.raises(ValueError):
        calls[call](kv=L.PagedKV(a["kv"].k_pool.transpose(0, 1), a["kv"].v_pool, a["kv"].stats, a["kv"].page_table, a["kv"].seq_lens))
    with pytest.raises(AttributeError):
        calls[call](kv=object())
    with pytest.raises(TypeError):
        B._native().decode(1, 2, 3)


def test_the_cache_is_described_as_through_ctypes():
    """A missing pool, a wrong number of heads, a bounded pool without its table: refused for the same reasons."""
    a, calls = _problem()
    kv = a["kv"]
    for bad in (L.PagedKV(None, kv.v_pool, kv.stats, kv.page_table, kv.seq_lens),
                L.PagedKV(kv.k_pool, kv.v_pool, kv.stats, kv.page_table, kv.seq_lens, pool_heads=3),
                L.PagedKV(kv.k_pool, kv.v_pool, kv.stats, kv.page_table, kv.seq_lens, k_pool_stream=kv.k_pool, v_pool_stream=kv.v_pool),
                L.PagedKV(kv.k_pool, kv.v_pool, kv.stats, kv.page_table, kv.seq_lens, kv_bits=5)):
        with pytest.raises(B.LserveError) as e:
            calls["decode"](kv=bad)
        assert e.value.code == -1
