"""Admission with many kv heads: counts of a call go over blocks of up to 16 heads, so head counts below, at and past that,
ones that leave a block with few heads, and ones that do not divide a block's threads.  Scores differ by head, tokens leave
from the ring and from the chunk; the state bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hk,W,P,chunks", [(15, 20, 16, [[40, 700], [600, 3]]), (16, 33, 4, [[513 + 33, 1]]), (17, 20, 16, [[700], [1200]]),
                                           (24, 8, 8, [[100, 0, 37], [530, 9, 8]]), (65, 16, 16, [[90, 640], [33, 15]]),
                                           (96, 16, 16, [[60, 300], [540, 7]]), (128, 40, 16, [[30, 200], [45, 600]])])
def test_many_heads(Hk, W, P, chunks):
    rng = np.random.default_rng(Hk)
    B = len(chunks[0])
    total = max(sum(c[s] for c in chunks) for s in range(B))
    max_gp = total // P + 2
    pair = Pair(1, Hk, Hk, 64, wg.BF16, P, W, B, max_gp, B * Hk * (max_gp + -(-W // P)), max_call_seqs=B,
                max_call_tokens=max(sum(c) for c in chunks))
    rates = list(np.clip(rng.beta(0.7, 1.5, Hk), 0.005, 0.995))
    for nt in chunks:
        k, v, g = rand_tokens(rng, sum(nt), Hk, 64, torch.bfloat16, rates=rates)
        pair.prefill(0, list(range(B)), nt, k, v, g, 0.5)
        pair.check_state()
