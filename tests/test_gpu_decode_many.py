"""Decode attention of more (sequence, kv head) units than the launch has blocks: even units, which waves take whole; units
of very different lengths, which waves share; long ones, which blocks share; empty ones in between; and page sizes below a
tile.  Every head against the oracle, twice the same bits, and the counters between the calls back at zero."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_q, rand_tokens

pytestmark = pytest.mark.gpu

EVEN, RAGGED = [0.3] * 8, [0.95, 0.01, 0.01, 0.1, 0.1, 0.1, 0.05, 0.2]


@pytest.mark.parametrize("dtype,d,G,P,B,W,T,rates", [
    (wg.BF16, 128, 4, 16, 36, 32, 90, EVEN),        # 288 units, a wave each
    (wg.BF16, 128, 4, 16, 128, 20, 60, EVEN),       # 1024 units: as many as waves
    (wg.BF16, 128, 4, 16, 64, 32, 900, RAGGED),     # shares of waves
    (wg.BF16, 128, 4, 32, 33, 32, 700, RAGGED),     # shares of blocks
    (wg.BF16, 64, 1, 4, 40, 16, 80, EVEN), (wg.BF16, 64, 8, 16, 48, 16, 500, RAGGED), (wg.BF16, 128, 8, 16, 64, 32, 600, RAGGED),
    (wg.BF16, 128, 2, 1, 34, 16, 60, EVEN), (wg.F32, 64, 4, 16, 64, 32, 400, RAGGED), (wg.F32, 128, 2, 16, 33, 16, 300, RAGGED),
    (wg.F32, 128, 8, 8, 40, 16, 60, EVEN)])
def test_more_units_than_blocks(dtype, d, G, P, B, W, T, rates):
    rng = np.random.default_rng(B * T + d)
    Hk, tdt = 8, torch.float32 if dtype == wg.F32 else torch.bfloat16
    lens = [0 if s % 9 == 4 else max(1, T - 7 * (s % 5)) for s in range(B)]  # some slots were never used
    pages = sum(Hk * (-(-n // P) + -(-W // P) + 1) for n in lens)
    pair = Pair(1, G * Hk, Hk, d, dtype, P, W, B, T // P + 2, pages, max_call_seqs=B, max_call_tokens=sum(lens))
    ids = list(range(B))
    k, v, g = rand_tokens(rng, sum(lens), Hk, d, tdt, rates=rates)
    pair.prefill(0, ids, lens, k, v, g, 0.5)
    q = rand_q(rng, B, G * Hk, d, tdt)
    used = [s for s in ids if lens[s] > 0]
    out, ref = pair.attend(0, ids, q)
    err = np.abs(out[used] - ref[used])
    assert (out[[s for s in ids if lens[s] == 0]] == 0).all()
    assert np.isfinite(out).all() and err.max() <= (2e-5 if dtype == wg.F32 else 1e-2) and err.mean() <= 1e-3, err.max()
    for _ in range(3):
        again, _ = pair.attend(0, ids, q)
        np.testing.assert_array_equal(again, out)
    lay = pair.pool.layout
    assert int(pair.pool.meta_buf[lay.unit_counters:lay.unit_counters + 4096].view(torch.int32).abs().sum()) == 0
    # a slot in the middle and the last one alone: the kernel of few units
    few = used[len(used) // 2:len(used) // 2 + 2]
    one, _ = pair.attend(0, few, q[few])
    assert np.abs(one - ref[few]).max() <= (2e-5 if dtype == wg.F32 else 1e-2)
