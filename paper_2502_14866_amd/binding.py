"""Binding of liblserve.so: argument marshalling only, every step runs in the HIP kernels.  The three calls of a decode step are
marshalled natively (csrc/py_calls.cpp), the others by ctypes."""
from __future__ import annotations

import contextlib
import ctypes
import os
import warnings
from dataclasses import dataclass
from typing import Optional, Sequence

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# LSERVE_LIBRARY points at another build of the same library (e.g. an instrumented one)
_LIB_PATH = os.environ.get("LSERVE_LIBRARY") or os.path.join(_HERE, "liblserve.so")
_lib = None
_calls = None

LSERVE_CALL_BUILD_PAGE_STATS = 0
LSERVE_CALL_SELECT_PAGES = 1
LSERVE_CALL_SPARSE_PREFILL = 2
LSERVE_CALL_SPARSE_DECODE = 3

EXPORTED_SYMBOLS = (
    "lserve_build_page_stats",
    "lserve_select_pages",
    "lserve_sparse_prefill",
    "lserve_sparse_decode",
    "lserve_append_kv",
    "lserve_sparse_prefill_masked",
    "lserve_sparse_prefill_paged",
    "lserve_sparse_prefill_chunk",
    "lserve_chunk_scratch_bytes",
    "lserve_paged_prefill_workspace_bytes",
    "lserve_masked_prefill_workspace_bytes",
    "BlockMask",
    "lserve_workspace_bytes",
    "lserve_strerror",
    "lserve_last_hip_error",
    "lserve_init",
    "lserve_sparse_decode_noalloc",
    "lserve_probe_decode_read",
    "lserve_probe_prefill_shape",
    "lserve_probe_prefill_plan",
    "lserve_probe_prefill_longest_first",
    "lserve_probe_mask_walk",
)


class LserveError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where} failed with code {code}: {lserve_strerror(code)}"
                         + (f" (hipError_t {lserve_last_hip_error()})" if code == -4 else ""))


class _CAttnDesc(ctypes.Structure):
    _fields_ = [
        ("num_q_heads", ctypes.c_int32), ("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
        ("page_size", ctypes.c_int32), ("logical_page_size", ctypes.c_int32), ("dtype", ctypes.c_int32),
        ("sink_tokens", ctypes.c_int32), ("local_tokens", ctypes.c_int32),
        ("kv_head_is_streaming", ctypes.POINTER(ctypes.c_uint8)), ("sm_scale", ctypes.c_float),
    ]


class _CPagedKV(ctypes.Structure):
    _fields_ = [
        ("k_pool", ctypes.c_void_p), ("v_pool", ctypes.c_void_p), ("stats", ctypes.c_void_p),
        ("page_table", ctypes.c_void_p), ("seq_lens", ctypes.c_void_p),
        ("batch", ctypes.c_int32), ("max_pages_per_seq", ctypes.c_int32), ("num_pages", ctypes.c_int32),
        ("pool_heads", ctypes.c_int32),
        ("k_pool_stream", ctypes.c_void_p), ("v_pool_stream", ctypes.c_void_p), ("ring_table", ctypes.c_void_p),
        ("num_pages_stream", ctypes.c_int32), ("kv_bits", ctypes.c_int32),
    ]


class _CBlockMask(ctypes.Structure):
    _fields_ = [
        ("head_mask", ctypes.c_void_p), ("q_tile_start", ctypes.c_void_p), ("row_ptr", ctypes.c_void_p),
        ("cols", ctypes.c_void_p),
        ("num_masks", ctypes.c_int32), ("rows_per_mask", ctypes.c_int32), ("nnz", ctypes.c_int32),
    ]


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """Load liblserve.so; raises if it has not been built (there is no fallback path)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(
                f"{_LIB_PATH} is missing: build it with `python -m paper_2502_14866_amd.build` "
                "(or __graft_entry__.build()); there is no CPU fallback")
        lib = ctypes.CDLL(_LIB_PATH)
        vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
        dp, kp = ctypes.POINTER(_CAttnDesc), ctypes.POINTER(_CPagedKV)
        lib.lserve_build_page_stats.argtypes = [dp, kp, vp, i32, vp]
        lib.lserve_select_pages.argtypes = [dp, kp, vp, i32, vp, vp, vp, vp, vp, vp, sz, vp]
        lib.lserve_sparse_prefill.argtypes = [dp, vp, vp, vp, vp, i32, i32, i32, vp, vp, vp, sz, vp]
        lib.lserve_sparse_decode.argtypes = [dp, kp, vp, vp, vp, vp, i32, vp, vp, vp, sz, vp]
        lib.lserve_append_kv.argtypes = [dp, kp, vp, vp, vp, vp, i32, vp]
        lib.lserve_append_kv.restype = ctypes.c_int
        mp = ctypes.POINTER(_CBlockMask)
        lib.lserve_sparse_prefill_masked.argtypes = [dp, mp, vp, vp, vp, vp, i32, i32, i32, vp, vp, vp, sz, vp]
        lib.lserve_sparse_prefill_masked.restype = ctypes.c_int
        lib.lserve_masked_prefill_workspace_bytes.argtypes = [dp, i32, i32, i32, i32, i32]
        lib.lserve_masked_prefill_workspace_bytes.restype = ctypes.c_size_t
        lib.lserve_sparse_prefill_paged.argtypes = [dp, kp, vp, vp, i32, i32, i32, vp, vp, vp, sz, vp]
        lib.lserve_sparse_prefill_paged.restype = ctypes.c_int
        lib.lserve_sparse_prefill_paged_scratch.argtypes = [dp, kp, vp, vp, i32, i32, i32, vp, vp, vp, sz, vp]
        lib.lserve_sparse_prefill_paged_scratch.restype = ctypes.c_int
        lib.lserve_sparse_prefill_chunk.argtypes = [dp, kp, vp, vp, vp, vp, i32, i32, vp, vp, vp]
        lib.lserve_sparse_prefill_chunk.restype = ctypes.c_int
        lib.lserve_sparse_prefill_chunk_scratch.argtypes = [dp, kp, vp, vp, vp, vp, i32, i32, vp, vp, vp, sz, vp]
        lib.lserve_sparse_prefill_chunk_scratch.restype = ctypes.c_int
        lib.lserve_chunk_scratch_bytes.argtypes = [dp, i32, i32, i32, i32, i32]
        lib.lserve_chunk_scratch_bytes.restype = sz
        lib.lserve_paged_prefill_workspace_bytes.argtypes = [dp, i32, i32]
        lib.lserve_paged_prefill_workspace_bytes.restype = ctypes.c_size_t
        lib.lserve_workspace_bytes.argtypes = [ctypes.c_int, dp, i32, i32, i32, i32]
        lib.lserve_workspace_bytes.restype = sz
        lib.lserve_strerror.argtypes = [ctypes.c_int]
        lib.lserve_strerror.restype = ctypes.c_char_p
        lib.lserve_last_hip_error.restype = ctypes.c_int
        lib.lserve_sparse_decode_noalloc.argtypes = [dp, kp, vp, vp, vp, vp, i32, vp, vp, vp]
        lib.lserve_sparse_decode_noalloc.restype = ctypes.c_int
        lib.lserve_probe_decode_read.argtypes = [dp, kp, vp, vp, vp, i32, vp]
        lib.lserve_probe_decode_read.restype = ctypes.c_int
        lib.lserve_probe_prefill_shape.argtypes = [dp, i32, i32, i32, i32, i32, ctypes.POINTER(i32)]
        lib.lserve_probe_prefill_shape.restype = ctypes.c_int
        lib.lserve_probe_prefill_plan.argtypes = [dp, i32, i32, i32, i32, i32, i32, ctypes.POINTER(i32)]
        lib.lserve_probe_prefill_plan.restype = ctypes.c_int
        lib.lserve_probe_prefill_longest_first.argtypes = [dp, i32, i32, i32, ctypes.POINTER(i32)]
        lib.lserve_probe_prefill_longest_first.restype = ctypes.c_int
        lib.lserve_probe_mask_walk.argtypes = [dp, i32, i32, i32, i32, i32, i32, ctypes.POINTER(i32)]
        lib.lserve_probe_mask_walk.restype = ctypes.c_int
        lib.lserve_init.argtypes = []
        lib.lserve_init.restype = ctypes.c_int
        for name in ("lserve_build_page_stats", "lserve_select_pages", "lserve_sparse_prefill",
                     "lserve_sparse_decode"):
            getattr(lib, name).restype = ctypes.c_int
        _lib = lib
    return _lib


class _CtypesCalls:
    """The native calls by ctypes, where the extension is not there or not of this torch; desc as its address."""

    @staticmethod
    def append(desc, kv, k_new, v_new, cu_new, start_pos, max_new_per_seq, stream):
        return load_library().lserve_append_kv(_CAttnDesc.from_address(desc), kv.c(), _ptr(k_new), _ptr(v_new), _ptr(cu_new),
                                               _ptr(start_pos), max_new_per_seq, stream)

    @staticmethod
    def select(desc, kv, q, budget_tokens, stats_valid_len, sel_pages, sel_count, sel_seq_len, scores_out, workspace, stream):
        ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
        return load_library().lserve_select_pages(_CAttnDesc.from_address(desc), kv.c(), _ptr(q), budget_tokens,
                                                  _ptr(stats_valid_len), _ptr(sel_pages), _ptr(sel_count), _ptr(sel_seq_len),
                                                  _ptr(scores_out), _ptr(workspace), ws_bytes, stream)

    @staticmethod
    def decode(desc, kv, q, sel_pages, sel_count, sel_seq_len, out, lse_out, workspace, stream):
        ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
        sel_stride = 0 if sel_pages is None else sel_pages.shape[-1]
        return load_library().lserve_sparse_decode(_CAttnDesc.from_address(desc), kv.c(), _ptr(q), _ptr(sel_pages),
                                                   _ptr(sel_count), _ptr(sel_seq_len), sel_stride, _ptr(out), _ptr(lse_out),
                                                   _ptr(workspace), ws_bytes, stream)


def _native():
    """The native calls, bound to the loaded library; without the extension (only the library was built, or it was built with another
    torch or Python) the same by ctypes, some five microseconds a call slower."""
    global _calls
    if _calls is None:
        lib = load_library()
        try:
            from . import _calls as calls

            if calls.torch_version != torch.__version__:
                raise ImportError(f"_calls was built with torch {calls.torch_version}, this is {torch.__version__}")
            calls.bind(*(ctypes.cast(f, ctypes.c_void_p).value
                         for f in (lib.lserve_append_kv, lib.lserve_select_pages, lib.lserve_sparse_decode)))
        except ImportError as e:
            warnings.warn(f"the binding's native calls are missing ({e}): decode steps are marshalled by ctypes; build them with "
                          "`python -m paper_2502_14866_amd.build` (or __graft_entry__.build())", RuntimeWarning, stacklevel=3)
            calls = _CtypesCalls
        _calls = calls
    return _calls


@dataclass
class AttnDesc:
    """Mirror of lserve_attn_desc."""
    num_q_heads: int
    num_kv_heads: int
    streaming_flags: Sequence[int]
    head_dim: int = 128
    page_size: int = 64
    logical_page_size: int = 16
    dtype: torch.dtype = torch.float16
    sink_tokens: int = 128
    local_tokens: int = 512
    sm_scale: float = 0.0

    def __post_init__(self):
        flags = [1 if f else 0 for f in self.streaming_flags]
        self._flags = (ctypes.c_uint8 * max(1, len(flags)))(*flags)
        self._c = _CAttnDesc(
            self.num_q_heads, self.num_kv_heads, self.head_dim, self.page_size, self.logical_page_size,
            {torch.float16: 0, torch.bfloat16: 1}.get(self.dtype, -1), self.sink_tokens, self.local_tokens,
            ctypes.cast(self._flags, ctypes.POINTER(ctypes.c_uint8)), float(self.sm_scale))

        self._address = ctypes.addressof(self._c)

    def c(self):
        return ctypes.byref(self._c)


@dataclass
class PagedKV:
    """Mirror of lserve_paged_kv; keeps the tensors alive."""
    k_pool: Optional[torch.Tensor]
    v_pool: Optional[torch.Tensor]
    stats: Optional[torch.Tensor]
    page_table: torch.Tensor
    seq_lens: torch.Tensor
    # two-way cache: heads per page of the main pool (0 = all KV heads) and the streaming heads' bounded pool
    pool_heads: int = 0
    k_pool_stream: Optional[torch.Tensor] = None
    v_pool_stream: Optional[torch.Tensor] = None
    ring_table: Optional[torch.Tensor] = None
    # 16: pools of the layer's 16-bit dtype [pages, heads, N_P, D]; 8 or 4: quantised pages, uint8
    # [pages, heads, 64 * D * kv_bits / 8 + 256]
    kv_bits: int = 16

    def c(self):
        sized = self.stats if self.stats is not None else self.v_pool if self.v_pool is not None else self.k_pool
        num_pages = 0 if sized is None else sized.size(0)
        num_pages_stream = 0 if self.k_pool_stream is None else self.k_pool_stream.size(0)
        self._c = _CPagedKV(_ptr(self.k_pool), _ptr(self.v_pool), _ptr(self.stats), _ptr(self.page_table),
                            _ptr(self.seq_lens), self.page_table.size(0), self.page_table.size(1), num_pages,
                            self.pool_heads, _ptr(self.k_pool_stream), _ptr(self.v_pool_stream),
                            _ptr(self.ring_table), num_pages_stream, self.kv_bits)
        return ctypes.byref(self._c)


# A decode step of a small batch is two or three calls of some ten microseconds of GPU work each, so the marshalling is kept to
# what a call cannot do without: addresses travel as plain integers (the argument types make pointers of them), the
# current stream is asked for as a handle, without the stream object around it, and the calls of the step itself are native.
def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    if t is None:
        return None
    if not t.is_contiguous():
        raise ValueError("lserve binding takes contiguous tensors")
    return t.data_ptr()


_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)  # private names: the public way where they are gone
_device = getattr(torch._C, "_cuda_getDevice", None)


def _stream(stream) -> int:
    if stream is None:
        if _raw_stream and _device and torch.cuda.is_initialized():
            return _raw_stream(_device())
        stream = torch.cuda.current_stream()
    return stream.cuda_stream if hasattr(stream, "cuda_stream") else int(stream)


def _check(rc: int, where: str) -> None:
    if rc:
        raise LserveError(rc, where)


def lserve_strerror(code: int) -> str:
    return load_library().lserve_strerror(int(code)).decode()


def lserve_last_hip_error() -> int:
    return int(load_library().lserve_last_hip_error())


def lserve_init() -> None:
    _check(load_library().lserve_init(), "lserve_init")


def lserve_workspace_bytes(which_call: int, desc: AttnDesc, batch: int = 0, max_pages_per_seq: int = 0,
                           sel_stride_or_budget_pages: int = 0, total_tokens: int = 0) -> int:
    return int(load_library().lserve_workspace_bytes(which_call, desc.c(), batch, max_pages_per_seq,
                                                     sel_stride_or_budget_pages, total_tokens))


def lserve_build_page_stats(desc: AttnDesc, kv: PagedKV, start_pos: Optional[torch.Tensor] = None,
                            max_tail_pages: int = 0, stream=None) -> None:
    _check(load_library().lserve_build_page_stats(desc.c(), kv.c(), _ptr(start_pos), max_tail_pages,
                                                  _stream(stream)), "lserve_build_page_stats")


def lserve_append_kv(desc: AttnDesc, kv: PagedKV, k_new: torch.Tensor, v_new: torch.Tensor, cu_new: torch.Tensor,
                     start_pos: torch.Tensor, max_new_per_seq: int, stream=None) -> None:
    _check((_calls or _native()).append(desc._address, kv, k_new, v_new, cu_new, start_pos, max_new_per_seq,
                                        _stream(stream)), "lserve_append_kv")


def lserve_select_pages(desc: AttnDesc, kv: PagedKV, q: torch.Tensor, budget_tokens: int,
                        sel_pages: torch.Tensor, sel_count: torch.Tensor, sel_seq_len: torch.Tensor,
                        scores_out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                        stream=None, stats_valid_len: Optional[torch.Tensor] = None) -> None:
    _check((_calls or _native()).select(desc._address, kv, q, budget_tokens, stats_valid_len, sel_pages, sel_count, sel_seq_len,
                                        scores_out, workspace, _stream(stream)), "lserve_select_pages")


def lserve_chunk_scratch_bytes(desc: AttnDesc, batch: int, total_new: int, max_new_per_seq: int, pages: int,
                               kv_bits: int = 16) -> int:
    return int(load_library().lserve_chunk_scratch_bytes(desc.c(), batch, total_new, max_new_per_seq, pages, kv_bits))


def _capture_has_a_pool() -> bool:
    """Under capture: do allocations come from a pool that the graph keeps (torch.cuda.graph), or from the one whose memory is handed
    on after the call and would be somebody else's when the graph is replayed (a capture begun by other means)?"""
    probe = torch.empty((16,), dtype=torch.uint8, device="cuda")
    for segment in torch.cuda.memory_snapshot():
        if segment["address"] <= probe.data_ptr() < segment["address"] + segment["total_size"]:
            return tuple(segment.get("segment_pool_id", (0, 0))) != (0, 0)
    return False


def _chunk_scratch(desc: AttnDesc, q: torch.Tensor, batch: int, max_new_per_seq: int, pages: int, kv_bits: int,
                   stream) -> Optional[torch.Tensor]:
    """Scratch for a call on chunks, from torch's allocator, which hands freed memory on in the order of the stream it was taken on:
    it is taken on the stream of the call."""
    need = lserve_chunk_scratch_bytes(desc, batch, q.shape[0], max_new_per_seq, pages, kv_bits)
    if need == 0 or not q.is_cuda:
        return None
    handle = _stream(stream)
    on_stream = contextlib.nullcontext()
    if handle != _stream(None):
        if isinstance(stream, torch.cuda.Stream):
            on_stream = torch.cuda.stream(stream)
        elif handle == 0:
            on_stream = torch.cuda.stream(torch.cuda.default_stream(q.device))
        elif handle < 16:  # the runtime's names for streams are not addresses, as which torch would take them
            return None
        else:
            on_stream = torch.cuda.stream(torch.cuda.ExternalStream(handle, device=q.device))
    with on_stream:
        if torch.cuda.is_current_stream_capturing() and not _capture_has_a_pool():
            return None
        try:
            return torch.empty((need,), dtype=torch.uint8, device="cuda")
        except torch.cuda.OutOfMemoryError:
            warnings.warn(f"no memory for the {need} bytes of scratch of a call on chunks: it goes without, which is slower and adds "
                          "up in another order; scratch= takes memory of the caller's, an empty tensor for none",
                          RuntimeWarning, stacklevel=3)
            return None


def lserve_sparse_prefill(desc: AttnDesc, q: torch.Tensor, k: torch.Tensor, v: torch.Tensor,
                          cu_seqlens: torch.Tensor, max_seqlen: int, out: torch.Tensor,
                          lse_out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                          stream=None) -> None:
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(load_library().lserve_sparse_prefill(desc.c(), _ptr(q), _ptr(k), _ptr(v), _ptr(cu_seqlens),
                                                cu_seqlens.shape[0] - 1, q.shape[0], max_seqlen, _ptr(out),
                                                _ptr(lse_out), _ptr(workspace), ws_bytes, _stream(stream)),
           "lserve_sparse_prefill")


@dataclass
class BlockMask:
    """Mirror of lserve_block_mask (device int32 tensors); keeps the tensors alive."""
    head_mask: torch.Tensor
    q_tile_start: torch.Tensor
    row_ptr: torch.Tensor
    cols: Optional[torch.Tensor]
    num_masks: int
    rows_per_mask: int

    @property
    def nnz(self) -> int:
        return 0 if self.cols is None else int(self.cols.numel())

    def c(self):
        self._c = _CBlockMask(_ptr(self.head_mask), _ptr(self.q_tile_start), _ptr(self.row_ptr), _ptr(self.cols),
                              self.num_masks, self.rows_per_mask, self.nnz)
        return ctypes.byref(self._c)


def lserve_masked_prefill_workspace_bytes(desc: AttnDesc, batch: int, total_tokens: int, max_seqlen: int,
                                          num_masks: int, nnz: int) -> int:
    return int(load_library().lserve_masked_prefill_workspace_bytes(desc.c(), batch, total_tokens, max_seqlen,
                                                                    num_masks, nnz))


def lserve_sparse_prefill_masked(desc: AttnDesc, mask: BlockMask, q: torch.Tensor, k: torch.Tensor, v: torch.Tensor,
                                 cu_seqlens: torch.Tensor, max_seqlen: int, out: torch.Tensor,
                                 lse_out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                                 stream=None) -> None:
    ws_bytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(load_library().lserve_sparse_prefill_masked(desc.c(), mask.c(), _ptr(q), _ptr(k), _ptr(v),
                                                       _ptr(cu_seqlens), cu_seqlens.shape[0] - 1, q.shape[0],
                                                       max_seqlen, _ptr(out), _ptr(lse_out), _ptr(workspace),
                                                       ws_bytes, _stream(stream)),
           "lserve_sparse_prefill_masked")


def lserve_paged_prefill_workspace_bytes(desc: AttnDesc, batch: int, max_pages_per_seq: int) -> int:
    return int(load_library().lserve_paged_prefill_workspace_bytes(desc.c(), batch, max_pages_per_seq))


def lserve_sparse_prefill_paged(desc: AttnDesc, kv: PagedKV, q: torch.Tensor, cu_q: torch.Tensor,
                                max_new_per_seq: int, max_seqlen: int, out: torch.Tensor,
                                lse_out: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None,
                                stream=None, scratch: Optional[torch.Tensor] = None) -> None:
    """workspace is not used.  scratch: see lserve_sparse_prefill_chunk; lserve_chunk_scratch_bytes with
    pages = min(page_table.shape[1], ceil(max_seqlen / 64))."""
    _ptr(workspace)  # unused, and contiguous all the same
    if scratch is None:
        pages = min(kv.page_table.shape[1], (max_seqlen - 1) // 64 + 1)
        scratch = _chunk_scratch(desc, q, cu_q.shape[0] - 1, max_new_per_seq, pages, 16, stream)
    _check(load_library().lserve_sparse_prefill_paged_scratch(
        desc.c(), kv.c(), _ptr(q), _ptr(cu_q), q.shape[0], max_new_per_seq, max_seqlen, _ptr(out), _ptr(lse_out), _ptr(scratch),
        0 if scratch is None else scratch.numel() * scratch.element_size(), _stream(stream)), "lserve_sparse_prefill_paged")


def lserve_sparse_prefill_chunk(desc: AttnDesc, kv: PagedKV, q: torch.Tensor, k_new: torch.Tensor, v_new: torch.Tensor,
                                cu_new: torch.Tensor, max_new_per_seq: int, out: torch.Tensor,
                                lse_out: Optional[torch.Tensor] = None, stream=None,
                                scratch: Optional[torch.Tensor] = None) -> None:
    """scratch: device memory of lserve_chunk_scratch_bytes(desc, batch, q.shape[0], max_new_per_seq, page_table.shape[1], kv_bits)
    bytes or more, not shared with work in flight; too little of it, an empty tensor for instance: the call does without.  None: taken
    from torch's allocator for the call (up to 1 GiB of expanded pages, by the width of the page table, and 34 to 136 MB of pieces),
    on whatever stream it goes to and from the graph's own pool under torch.cuda.graph, so that the same call gives the same bits
    everywhere.  A call goes without, slower and with sums in another order, where torch is out of memory (a RuntimeWarning says
    so) and in a capture begun by other means than torch.cuda.graph."""
    if scratch is None:
        scratch = _chunk_scratch(desc, q, cu_new.shape[0] - 1, max_new_per_seq, kv.page_table.shape[1], kv.kv_bits, stream)
    _check(load_library().lserve_sparse_prefill_chunk_scratch(
        desc.c(), kv.c(), _ptr(q), _ptr(k_new), _ptr(v_new), _ptr(cu_new), q.shape[0], max_new_per_seq, _ptr(out),
        _ptr(lse_out), _ptr(scratch), 0 if scratch is None else scratch.numel() * scratch.element_size(), _stream(stream)),
        "lserve_sparse_prefill_chunk")


def lserve_sparse_decode(desc: AttnDesc, kv: PagedKV, q: torch.Tensor, sel_pages: Optional[torch.Tensor],
                         sel_count: Optional[torch.Tensor], sel_seq_len: Optional[torch.Tensor],
                         out: torch.Tensor, lse_out: Optional[torch.Tensor] = None,
                         workspace: Optional[torch.Tensor] = None, stream=None) -> None:
    _check((_calls or _native()).decode(desc._address, kv, q, sel_pages, sel_count, sel_seq_len, out, lse_out, workspace,
                                        _stream(stream)), "lserve_sparse_decode")


def lserve_sparse_decode_noalloc(desc: AttnDesc, kv: PagedKV, q: torch.Tensor, sel_pages: Optional[torch.Tensor],
                                 sel_count: Optional[torch.Tensor], sel_seq_len: Optional[torch.Tensor],
                                 out: torch.Tensor, lse_out: Optional[torch.Tensor] = None, stream=None) -> None:
    sel_stride = 0 if sel_pages is None else sel_pages.shape[-1]
    _check(load_library().lserve_sparse_decode_noalloc(desc.c(), kv.c(), _ptr(q), _ptr(sel_pages), _ptr(sel_count),
                                                       _ptr(sel_seq_len), sel_stride, _ptr(out), _ptr(lse_out),
                                                       _stream(stream)), "lserve_sparse_decode_noalloc")


def lserve_probe_decode_read(desc: AttnDesc, kv: PagedKV, sel_pages: Optional[torch.Tensor],
                             sel_count: Optional[torch.Tensor], sel_seq_len: Optional[torch.Tensor], stream=None) -> None:
    sel_stride = 0 if sel_pages is None else sel_pages.shape[-1]
    _check(load_library().lserve_probe_decode_read(desc.c(), kv.c(), _ptr(sel_pages), _ptr(sel_count), _ptr(sel_seq_len),
                                                   sel_stride, _stream(stream)), "lserve_probe_decode_read")


def lserve_probe_prefill_shape(desc: AttnDesc, batch: int, total_rows: int, max_rows: int, pages: int = 0,
                               kv_bits: int = 16) -> tuple:
    """(key slices, dense heads folded, streaming heads folded, units are query tiles of one head) of a prefill launch."""
    shape = (ctypes.c_int32 * 4)()
    _check(load_library().lserve_probe_prefill_shape(desc.c(), batch, total_rows, max_rows, pages, kv_bits, shape),
           "lserve_probe_prefill_shape")
    return tuple(shape)


def lserve_probe_prefill_plan(desc: AttnDesc, batch: int, total_rows: int, max_rows: int, pages: int = 0, kv_bits: int = 16,
                              scratch: bool = True) -> dict:
    """The rest of it: key ranges of a dense and of a streaming head's rows, half workgroups, pieces, streaming heads in the launch
    that puts pieces together, expanded pages."""
    plan = (ctypes.c_int32 * 6)()
    _check(load_library().lserve_probe_prefill_plan(desc.c(), batch, total_rows, max_rows, pages, kv_bits, int(scratch), plan),
           "lserve_probe_prefill_plan")
    return dict(zip(("dense", "streaming", "half", "pieces", "apart", "expand"), plan))


def lserve_probe_prefill_longest_first(desc: AttnDesc, batch: int, total_rows: int, max_rows: int) -> bool:
    """Prompts: has the first workgroup of every compute unit, with the longest walks, the higher wave priority?"""
    first = ctypes.c_int32()
    _check(load_library().lserve_probe_prefill_longest_first(desc.c(), batch, total_rows, max_rows, ctypes.byref(first)),
           "lserve_probe_prefill_longest_first")
    return bool(first.value)


def lserve_probe_mask_walk(desc: AttnDesc, batch: int, total_tokens: int, max_seqlen: int, num_masks: int, rows_per_mask: int,
                           nnz: int) -> int:
    """How a masked prefill walks its lists: 0 merged, 1 by rows in four key slices, 2 by rows in half workgroups."""
    walk = ctypes.c_int32()
    _check(load_library().lserve_probe_mask_walk(desc.c(), batch, total_tokens, max_seqlen, num_masks, rows_per_mask, nnz,
                                                 ctypes.byref(walk)), "lserve_probe_mask_walk")
    return walk.value
