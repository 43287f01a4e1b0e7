"""Chunked prefill, in both of its forms (the grid's size decides), at the
edges of its 32-token stages, its three LDS slots, its 32-row tiles and
128-row workgroups: contexts and chunks around
multiples of them, chunks that start inside a stage and inside a block, one,
two, three and eight KV heads.  Poison past every context; every output row
against the oracle under the parity gate."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import compare, extend_attention  # noqa: E402
from test_gpu_extend import gpu_extend, make_extend  # noqa: E402

CASES = [
    # (contexts, chunks): chunk rows see the tokens up to their own position
    ([1, 2, 15, 16, 17, 31, 32, 33, 47, 48], [1, 1, 15, 16, 1, 31, 32, 33, 7, 8]),
    ([63, 64, 65, 95, 96, 97, 127, 128, 129], [63, 1, 65, 9, 32, 31, 127, 128, 33]),
    ([191, 192, 193, 287, 288, 289, 400], [1, 17, 193, 15, 16, 65, 64]),
    ([700, 1056, 640], [33, 1, 129]),
    # large enough a grid for the 128-row form at 64 heads over 8
    ([129, 96, 31, 64, 65, 200, 192, 33, 97, 1], [129, 64, 31, 63, 65, 100, 97, 32, 96, 1]),
]


@pytest.mark.parametrize("hq,hkv", [(4, 1), (16, 2), (12, 3), (64, 8)])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_extend_stage_edges(case, hq, hkv):
    ctx, chunk = CASES[case]
    print(f"[gpu case] extend stage edges Hq={hq} Hkv={hkv} ctx={ctx} chunk={chunk}", flush=True)
    w, q, q_start = make_extend(600 + 10 * case, ctx, chunk, hq=hq, hkv=hkv, poison=True)
    out = gpu_extend(w, q, q_start)
    ref, _ = extend_attention(q, q_start, w.k_pool, w.v_pool, w.block_tables, w.context_lens, w.scale)
    rep = compare(out, ref)
    assert rep.passed, f"{rep}"
