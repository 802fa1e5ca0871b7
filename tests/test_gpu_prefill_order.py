"""Prompts by half workgroups whose blocks are found in ragged batches of up to sixteen sequences, and those whose longest walk goes
first: sampled rows against the oracle, every row written."""
import pytest

import test_gpu_prefill_shapes as shapes
from workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("heads,kv_heads,lengths,first", [
    (64, 8, (1, 1300), 0),                                       # two sequences; one row
    (64, 8, (640, 640, 641), 0),                                 # levels that two or three of them share
    (64, 8, (64, 128, 192, 1, 63, 65, 2000, 127), 0),            # whole tiles and one off
    (32, 16, tuple(1 + 97 * i for i in range(15)), 0),
    (32, 8, (3001,) + tuple(7 + (311 * i) % 500 for i in range(15)), 0),   # sixteen: one long among short ones
    (32, 8, (77,) * 15 + (2500,), 0),                            # the long one last
    (32, 8, tuple(20 + (53 * i) % 700 for i in range(17)), 0),   # one more
    # the longest walk decides
    (32, 8, (4000,), 1),
    (32, 32, (3500,), 1),
    (32, 16, (200, 4300), 1),
    # and the same with a workgroup more to a unit than that
    (32, 8, (4700,), 0),
    (32, 16, (400, 4300), 0),
])
def test_blocks_of_ragged_batches(dtype, heads, kv_heads, lengths, first):
    import oracle
    import numpy as np
    import paper_2502_14866_amd as L

    w = Workload(name="order", batch=len(lengths), num_q_heads=heads, num_kv_heads=kv_heads, dtype=dtype,
                 streaming_kv_heads=tuple(range(kv_heads // 2)), sink_tokens=128, local_tokens=512, seed=29)
    desc = L.AttnDesc(heads, kv_heads, w.streaming_flags(), dtype=w.torch_dtype)
    assert L.lserve_probe_prefill_plan(desc, len(lengths), sum(lengths), max(lengths))["half"] == 1
    assert L.lserve_probe_prefill_longest_first(desc, len(lengths), sum(lengths), max(lengths)) == first
    pin, out, lse, _ = shapes._run(w, lengths)
    tok = shapes._sample(lengths, 3, 5)
    t, h = np.repeat(tok, heads), np.tile(np.arange(heads, dtype=np.int32), len(tok))
    ref, lse_ref = oracle.sparse_prefill_rows(pin.q, pin.k, pin.v, pin.cu_seqlens, w.streaming_flags(), 64, w.sink_tokens,
                                              w.local_tokens, t, h)
    shapes._check(w, lengths, pin, out, lse, ref, lse_ref, tok, f"order {dtype} {heads}/{kv_heads} {len(lengths)} sequences")
