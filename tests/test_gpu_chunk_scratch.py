"""Where the scratch of a call on chunks comes from: the same call has the same bits on every stream, eager and in a graph, unless the
caller declines scratch or there is none to be had."""
import ctypes
import warnings

import pytest
import torch

pytestmark = pytest.mark.gpu

N, NEW = 20000, 100  # long enough that dense walks are cut into pieces with scratch


@pytest.fixture(scope="module")
def problem():
    import paper_2502_14866_amd as L

    L.load_library()
    L.lserve_init()
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(17)
    rnd = lambda *s: torch.randn(s, generator=g, device=dev).to(torch.float16)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    pages = -(-(N + NEW) // 64)
    k, v = rnd(pages, 8, 64, 128), rnd(pages, 8, 64, 128)
    kv = L.PagedKV(k, v, None, torch.randperm(pages, generator=g, device=dev).to(torch.int32).reshape(1, -1), i32([N]))
    desc = L.AttnDesc(32, 8, [1, 1, 1, 1, 0, 0, 0, 0])
    q, kn, vn, cu = rnd(NEW, 32, 128), rnd(NEW, 8, 128), rnd(NEW, 8, 128), i32([0, NEW])

    class Problem:
        need = L.lserve_chunk_scratch_bytes(desc, 1, NEW, NEW, pages)
        none = torch.empty((0,), dtype=torch.uint8, device=dev)

        @staticmethod
        def chunk(out, **kw):
            L.lserve_sparse_prefill_chunk(desc, kv, q, kn, vn, cu, NEW, out, **kw)

        @staticmethod
        def paged(out, **kw):
            L.lserve_sparse_prefill_paged(desc, kv, q, cu, NEW, N, out, **kw)

        @staticmethod
        def new():
            return torch.full_like(q, float("nan"))
    p = Problem()
    assert p.need > 0
    for call in ("chunk", "paged"):
        with_scratch, without = p.new(), p.new()
        getattr(p, call)(with_scratch)
        getattr(p, call)(without, scratch=p.none)
        torch.cuda.synchronize()
        assert not torch.equal(with_scratch, without)  # or nothing below tells one from the other
        setattr(p, call + "_with", with_scratch)
        setattr(p, call + "_without", without)
    return p


@pytest.mark.parametrize("call", ["chunk", "paged"])
def test_every_stream_has_the_bits_of_the_current_one(problem, call):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    streams = [torch.cuda.current_stream(), torch.cuda.current_stream().cuda_stream, side, side.cuda_stream]
    outs = []
    for s in streams * 2:
        outs.append(problem.new())
        side.wait_stream(torch.cuda.current_stream())
        getattr(problem, call)(outs[-1], stream=s)
    with torch.cuda.stream(side):
        outs.append(problem.new())
        getattr(problem, call)(outs[-1])
        outs.append(problem.new())
        torch.cuda.default_stream().wait_stream(side)
        getattr(problem, call)(outs[-1], stream=0)
    torch.cuda.synchronize()
    assert all(torch.equal(o, getattr(problem, call + "_with")) for o in outs)


@pytest.mark.parametrize("call", ["chunk", "paged"])
def test_a_graph_has_the_bits_of_the_eager_call(problem, call):
    out, eager = problem.new(), problem.new()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        getattr(problem, call)(out)
        getattr(problem, call)(out)  # the second call's scratch may be the first's
    for i in range(4):
        out.fill_(float("nan"))
        getattr(problem, call)(eager)
        junk = torch.full((problem.need // 4,), float("inf"), device=out.device)  # whoever gets freed memory next
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, getattr(problem, call + "_with")) and torch.equal(eager, out), i
        del junk


def test_a_capture_without_a_pool_goes_without_scratch(problem):
    """Begun in the runtime, not by torch.cuda.graph: memory from torch's allocator would be handed on while the graph keeps its address."""
    import paper_2502_14866_amd as L

    hip = ctypes.CDLL(L.library_path())  # and what it is linked with
    side, out, eager = torch.cuda.Stream(), problem.new(), problem.new()
    torch.cuda.synchronize()
    graph, run = ctypes.c_void_p(), ctypes.c_void_p()
    s = ctypes.c_void_p(side.cuda_stream)
    with torch.cuda.stream(side):
        assert hip.hipStreamBeginCapture(s, ctypes.c_int(1)) == 0  # thread-local
        try:
            problem.chunk(out)
        finally:
            assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        out.fill_(float("nan"))
        problem.chunk(eager)
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(run, s) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, problem.chunk_without)
    assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0


@pytest.mark.parametrize("call", ["chunk", "paged"])
def test_scratch_of_the_callers(problem, call):
    for size, want in ((problem.need, "_with"), (problem.need + 4096, "_with"), (problem.need - 16, "_without"), (0, "_without")):
        out, scratch = problem.new(), torch.full((size + 256,), 0xff, dtype=torch.uint8, device="cuda")
        getattr(problem, call)(out, scratch=scratch[:size])
        torch.cuda.synchronize()
        assert torch.equal(out, getattr(problem, call + want))
        assert (scratch[size:] == 0xff).all()


def test_out_of_memory_is_said(problem, monkeypatch):
    empty, out = torch.empty, problem.new()

    def short(size, **kw):
        if size == (problem.need,):
            raise torch.cuda.OutOfMemoryError("none left")
        return empty(size, **kw)
    monkeypatch.setattr(torch, "empty", short)
    with pytest.warns(RuntimeWarning, match="scratch"):
        problem.chunk(out)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        problem.chunk(out, scratch=problem.none)  # declined: nothing to say
    torch.cuda.synchronize()
    assert torch.equal(out, problem.chunk_without)
