"""Write-back of rows with infinities and not-a-numbers: codes, scales, zero points and statistics.

A not-a-number takes no part in a row's range or in a channel's statistics (as with fminf and fmaxf), an infinite one saturates:
the expected bytes come from numpy in fp32, step by step, since the oracle's quantiser is for finite rows."""
import numpy as np
import pytest
import torch

from test_gpu_quant import _unpack_rows

pytestmark = pytest.mark.gpu

INF = float("inf")
SIGNALLING = {"fp16": 0x7d01, "bf16": 0x7fa1}  # quiet bit clear


def _rows(dtype):
    """[n, 128] rows of a token and head, and their bits as they go into the tensor."""
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    g = torch.Generator().manual_seed(3)
    plain = lambda: torch.randn((128,), generator=g) * 3
    rows = []

    def row(**at):
        x = plain() if at.pop("base", None) is None else torch.zeros(128)
        for where, v in at.items():
            x[int(where[1:])] = v
        rows.append(x)
    row()
    rows.append(torch.full((128,), -INF))
    rows.append(torch.full((128,), INF))
    row(_5=-INF)
    row(_127=INF)
    row(_0=-INF, _77=INF)
    row(_9=INF, _10=float("nan"), _11=-INF)
    row(_0=float("nan"))
    row(_64=float("nan"))
    rows.append(torch.full((128,), float("nan")))
    x = torch.full((128,), -INF)
    x[::2] = float("nan")
    rows.append(x)
    return torch.stack(rows).to(dt)


def _expected(x, bits):
    """Codes, scale and zero bits of rows x (fp32 [n, 128])."""
    top, big = np.float32(2 ** bits - 1), np.float32(65504)
    with np.errstate(all="ignore"):
        lo, hi = np.fmin.reduce(x, axis=1), np.fmax.reduce(x, axis=1)
        zero = np.fmin(np.fmax(lo, -big), big).astype(np.float16)
        zf = zero.astype(np.float32)
        scale = np.fmin((hi - zf) / top, big).astype(np.float16)
        sf = scale.astype(np.float32)[:, None]
        t = np.rint((x - zf[:, None]) / sf)
        codes = np.where(sf > 0, np.fmin(np.fmax(t, 0), top), 0).astype(np.uint8)
    return codes, scale, zero


def _append(x, bits, dtype, one_by_one):
    """Rows x [n, 128] as K and V of one KV head, written in one call or token by token; (pools, stats)."""
    import paper_2502_14866_amd as L

    L.load_library()
    dev = torch.device("cuda:0")
    n, dt = x.shape[0], x.dtype
    desc = L.AttnDesc(1, 1, [0], dtype=dt, sink_tokens=64, local_tokens=64)
    shape = (1, 1, 64, 128) if bits == 16 else (1, 1, 64 * 128 * bits // 8 + 256)
    k = torch.zeros(shape, dtype=dt if bits == 16 else torch.uint8, device=dev)
    v = torch.zeros_like(k)
    stats = torch.zeros((1, 1, 4, 2, 128), dtype=dt, device=dev)
    i32 = lambda *a: torch.tensor(a, dtype=torch.int32, device=dev)
    kv = L.PagedKV(k, v, stats, i32(0).reshape(1, 1), i32(n), kv_bits=bits)
    rows = x.reshape(n, 1, 128).to(dev)
    for at, m in ((i, 1) for i in range(n)) if one_by_one else ((0, n),):
        new = rows[at:at + m].clone()
        L.lserve_append_kv(desc, kv, new, new, i32(0, m), i32(at), m)
    torch.cuda.synchronize()
    return k.cpu(), v.cpu(), stats.cpu()


def _check(x, bits, dtype, one_by_one):
    k, v, stats = _append(x, bits, dtype, one_by_one)
    n, f = x.shape[0], x.float().numpy()
    if bits == 16:
        assert torch.equal(k.view(torch.int16)[0, 0, :n], x.view(torch.int16)) and torch.equal(v.view(torch.int16), k.view(torch.int16))
    else:
        codes, scale, zero = _expected(f, bits)
        for pool in (k, v):
            raw, tail = pool.numpy()[0, 0], 64 * 128 * bits // 8
            sz = np.ascontiguousarray(raw[tail:]).view(np.float16).reshape(64, 2)[:n]
            assert np.array_equal(sz[:, 0].view(np.uint16), scale.view(np.uint16)), (sz[:, 0], scale)
            assert np.array_equal(sz[:, 1].view(np.uint16), zero.view(np.uint16)), (sz[:, 1], zero)
            got = _unpack_rows(raw[:tail].reshape(64, 128 * bits // 8), bits)[:n]
            assert np.array_equal(got, codes), np.argwhere(got != codes)[:8]
    for page in range(-(-n // 16)):
        part = f[16 * page:16 * page + 16]
        with np.errstate(all="ignore"):
            want = np.fmax(np.fmax.reduce(part, axis=0), -INF), np.fmin(np.fmin.reduce(part, axis=0), INF)
        for side in (0, 1):
            assert np.array_equal(stats[0, 0, page, side].float().numpy(), want[side].astype(np.float32)), (page, side)


@pytest.mark.parametrize("one_by_one", [False, True])
@pytest.mark.parametrize("bits", [16, 8, 4])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_rows_with_infinities_and_not_a_numbers(dtype, bits, one_by_one):
    _check(_rows(dtype), bits, dtype, one_by_one)


@pytest.mark.parametrize("one_by_one", [False, True])
@pytest.mark.parametrize("dtype,bits", [("fp16", 16), ("fp16", 8), ("fp16", 4), ("bf16", 16)])
def test_signalling_not_a_numbers_do_not_drop_what_came_before(dtype, bits, one_by_one):
    """The extremes of a row in front of one in the same lane, those of a channel in rows above one."""
    x = torch.randn((23, 128), generator=torch.Generator().manual_seed(8)).to(_rows(dtype).dtype)
    x[0, 40], x[0, 41], x[3, 8], x[3, 9], x[5, 126], x[2, :] = -50.0, 60.0, -70.0, 80.0, 90.0, -33.0
    raw = x.view(torch.int16)
    for r, c in [(0, 42), (0, 43), (3, 10), (3, 15), (5, 127), (6, 7), (16, 100), (20, 100)] + [(6, c) for c in range(64, 96)]:
        raw[r, c] = SIGNALLING[dtype] if c % 2 else SIGNALLING[dtype] - 0x8000
    raw[22] = SIGNALLING[dtype]
    _check(x, bits, dtype, one_by_one)
