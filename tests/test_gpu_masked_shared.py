"""Masked prefill by half workgroups, of which two heads of a group share one if they have a mask in common, by key slices and by
merged lists.  Masks given to the heads of a group in every way, streaming groups with listed masks, groups of odd size, against the
oracle."""
import numpy as np
import pytest
import torch

import oracle
from workloads import Workload

from test_gpu_prefill_shapes import HALVES, MERGED, SLICES, _check, _run, _sample

pytestmark = pytest.mark.gpu

ROWS = {
    "few": lambda b, i: [j for j in range(i + 1) if (7 * j + 3 * i) % 5 == 0 or j == i],
    "other": lambda b, i: [j for j in range(i + 1) if (j + i) % 3 == 0],  # the diagonal tile is kept by some rows only
    "gaps": lambda b, i: [] if i % 4 == 3 else [j for j in range(i + 1) if j % 2 == 0 or j == i],  # rows that keep nothing
    "most": lambda b, i: [j for j in range(i + 1) if (j + 2 * i) % 7 or j == i],
    "holes": lambda b, i: [] if i % 5 == 3 else [j for j in range(i + 1) if (j + i) % 9],  # the same, and diagonals left out
    "all": lambda b, i: list(range(i + 1)),
}
SOME = [1] * 5 + [-1] * 11 + [0, 0, 0, 1, 1, 0, 1, 1, -1, 0, 1, -1, 0, 0, 0, 0]
ONE_OR_NONE = [-1, 0, 0, -1, 0, 0, 0, 0, 0, -1, -1, -1, -1, 0, -1, 0]  # one mask or none


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,lengths,masks,head_mask,walk", [
    (32, 8, (1500, 333), ("few", "other"), [-1] * 16 + [0, 1, 0, 1] * 4, HALVES),  # two pairs, heads in turn
    (32, 8, (1999,), ("few", "gaps"), SOME, SLICES),
    (32, 8, (2600,), ("few", "gaps"), SOME, HALVES),
    (16, 4, (1000, 65, 1), ("gaps",), ONE_OR_NONE, SLICES),
    (16, 4, (12000, 65, 1), ("gaps",), ONE_OR_NONE, HALVES),
    (64, 8, (1300,), ("few", "other", "gaps"), [(5 * h + h // 7) % 4 - 1 for h in range(64)], HALVES),    # four pairs to a group
    (24, 4, (2100, 700), ("other", "few", "gaps"), [(h * h) % 3 for h in range(24)], SLICES),  # three, listed masks on streaming heads
    (24, 4, (7000, 700), ("other", "few", "gaps"), [(h * h) % 3 for h in range(24)], HALVES),
    (24, 8, (2500, 70), ("few",), [-1] * 7 + [0] * 17, SLICES),                                    # three heads to a group
    (24, 8, (5000, 70), ("few",), [-1] * 7 + [0] * 17, HALVES),
    (4, 2, (3100,), ("few",), [0, 0, 0, 0], SLICES),
    # lists of most tiles, by blocks of four query tiles: whole blocks, remainders, rows that keep nothing, masks of every kind in a group
    (32, 8, (3001, 500), ("most", "holes", "all"), [h % 4 - 1 for h in range(32)], MERGED),
    (24, 8, (5000, 333, 1), ("most", "holes"), [(h * h) % 3 - 1 for h in range(24)], MERGED),
    (64, 8, (2048, 64), ("most", "holes", "all"), [(5 * h + h // 7) % 4 - 1 for h in range(64)], MERGED),
    (16, 8, (9000,), ("most", "holes"), [h % 2 for h in range(16)], MERGED),
])
def test_two_heads_to_a_row(dtype, heads, kv_heads, lengths, masks, head_mask, walk):
    w = Workload(name="shared", batch=len(lengths), num_q_heads=heads, num_kv_heads=kv_heads, dtype=dtype,
                 streaming_kv_heads=tuple(range(kv_heads // 2)), sink_tokens=64, local_tokens=256, seed=61)
    pin, out, lse, (qts, rp, cl, rows) = _run(w, lengths, [ROWS[m] for m in masks], head_mask, past_diagonal=3, walk=walk)
    tok = _sample(lengths, 30, 11)
    t, h = np.repeat(tok, heads), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.block_mask_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64,
                                                  w.sink_tokens, w.local_tokens, head_mask, qts, rp, cl, rows, t, h)
    # rows that keep nothing: 0 and -inf on both sides (and out of the comparison of finite numbers)
    at = torch.from_numpy(tok).long().to(out.device)
    none = torch.from_numpy(np.isneginf(lse_ref.reshape(len(tok), heads))).to(out.device)
    assert (lse.t()[at][none] == -np.inf).all() and (out[at][none] == 0).all() and torch.isfinite(lse.t()[at][~none]).all()
    if none.any():
        lse[:, at] = torch.where(none.t(), torch.zeros_like(lse[:, at]), lse[:, at])
        lse_ref = np.where(np.isneginf(lse_ref), 0.0, lse_ref)
    _check(w, lengths, pin, out, lse, ref, lse_ref, tok, f"masked prefill {dtype} {heads}/{kv_heads}")
