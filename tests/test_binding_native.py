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


def _captured(monkeypatch, route):
    """What the three entry points of the library are handed, natively or by ctypes: plain values, structs as bytes."""
    import ctypes
    import types

    a, _ = _problem()
    kv = L.PagedKV(a["kv"].k_pool, a["kv"].v_pool, a["kv"].stats, a["kv"].page_table, a["kv"].seq_lens, pool_heads=1,
                   k_pool_stream=a["kv"].k_pool[:5], v_pool_stream=a["kv"].v_pool[:5], ring_table=a["kv"].page_table, kv_bits=8)
    vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    dp, kp = ctypes.POINTER(B._CAttnDesc), ctypes.POINTER(B._CPagedKV)
    types_of = {"lserve_append_kv": [dp, kp, vp, vp, vp, vp, i32, vp], "lserve_select_pages": [dp, kp, vp, i32, vp, vp, vp, vp, vp, vp, sz, vp],
                "lserve_sparse_decode": [dp, kp, vp, vp, vp, vp, i32, vp, vp, vp, sz, vp]}
    seen, lib = [], types.SimpleNamespace()
    for name, arg_types in types_of.items():
        def body(desc, cache, *rest, name=name):
            seen.append((name, bytes(desc.contents), B._CPagedKV.from_buffer_copy(cache.contents), *rest))
            return 0
        stub = ctypes.CFUNCTYPE(ctypes.c_int, *arg_types)(body)
        setattr(lib, name, stub)
    monkeypatch.setattr(B, "_lib", lib)
    monkeypatch.setattr(B, "_calls", None)
    if route == "native":
        B._native()
    else:
        monkeypatch.setattr(B, "_calls", B._CtypesCalls)
    ws = torch.zeros((3, 8), dtype=torch.float32)
    big = 2 ** 70 + 5  # wraps
    L.lserve_append_kv(a["desc"], kv, a["new"], a["new"], a["cu"], a["ssl"], 7, 0x1230)
    L.lserve_select_pages(a["desc"], kv, a["q"], big, a["sel"], a["cnt"], a["ssl"], None, ws, 0, a["ssl"])
    L.lserve_sparse_decode(a["desc"], kv, a["q"], a["sel"], a["cnt"], a["ssl"], a["q"], None, ws, 0)
    L.lserve_sparse_decode(a["desc"], kv, a["q"], None, None, None, a["q"], None, None, 0)
    monkeypatch.undo()
    if route == "native":  # back to the library itself
        lib = B.load_library()
        B._native().bind(*(ctypes.cast(getattr(lib, f), vp).value for f in types_of))
    base = {t.data_ptr(): k for k, t in list(a.items()) + [("ws", ws)] if isinstance(t, torch.Tensor)}
    return [tuple(base.get(x, x) if isinstance(x, int) else x for x in (s[0], *s[3:])) for s in seen], [s[1][:32] for s in seen], \
        [s[2] for s in seen]


def test_both_routes_hand_over_the_same(monkeypatch):
    native, ctyped = _captured(monkeypatch, "native"), _captured(monkeypatch, "ctypes")
    assert native[0] == ctyped[0] and native[1] == ctyped[1] and len(native[0]) == 4
    for x, y in zip(native[2], ctyped[2]):
        for field, kind in B._CPagedKV._fields_:
            assert (getattr(x, field) is None) == (getattr(y, field) is None), field
            if kind is not B.ctypes.c_void_p:
                assert getattr(x, field) == getattr(y, field), field


@pytest.mark.parametrize("broken", ["missing", "another torch"])
def test_without_the_extension_calls_go_by_ctypes(monkeypatch, broken):
    """Only the library was built, or the extension is of another torch: said once, and refused is what was refused."""
    import sys
    import types

    import paper_2502_14866_amd

    module = None if broken == "missing" else types.SimpleNamespace(torch_version="0.0.0")
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setitem(sys.modules, "paper_2502_14866_amd._calls", module)
    if module is None:
        monkeypatch.delattr(paper_2502_14866_amd, "_calls", raising=False)
    else:
        monkeypatch.setattr(paper_2502_14866_amd, "_calls", module, raising=False)
    _, calls = _problem()
    with pytest.warns(RuntimeWarning, match="native calls"):
        with pytest.raises(B.LserveError) as e:
            calls["append"]()
    assert e.value.code == -1
    for call, code in (("select", -3), ("decode", -3)):
        with pytest.raises(B.LserveError) as e:
            calls[call]()
        assert e.value.code == code
    with pytest.raises(ValueError):
        calls["decode"](q=torch.zeros((2, 128, 4), dtype=torch.float16).transpose(1, 2))
