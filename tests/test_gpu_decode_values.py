"""Decode attention of bf16 pools with values of V at the end of the range."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_tokens

pytestmark = pytest.mark.gpu

SHAPES = [(128, 4), (128, 1), (128, 2), (128, 8), (64, 4), (64, 1), (64, 2), (64, 8)]


@pytest.mark.parametrize("d,G", SHAPES)
@pytest.mark.parametrize("B,Hk", [(12, 2), (40, 8)], ids=["one-unit-a-block", "many-units"])
def test_large_values_under_a_rising_score(d, G, B, Hk):
    """A later key's score is 7.8 powers of two above all others' and its values are 1e38: the weighted sum is finite."""
    rng = np.random.default_rng(d + G)
    n, W, P = 240, 16, 16  # 15 tiles: two pairs a wave where a block has the unit, eight where a wave has it
    pair = Pair(1, G * Hk, Hk, d, wg.BF16, P, W, B, n // P + 2, B * Hk * (n // P + 3), max_call_seqs=B, max_call_tokens=B * n)
    k = torch.zeros((B, n, Hk, d), dtype=torch.bfloat16)
    v = 1e35 * torch.from_numpy(rng.standard_normal((B, n, Hk, d)).astype(np.float32))
    for b in range(B):
        at = (14 * (b % 12) + 70) % n
        k[b, at, :, 0] = 5.4375  # 7.84 powers of two with a query of one
        v[b, at] = 1e38 * torch.from_numpy(np.where(rng.random((Hk, d)) < 0.5, -1, 1).astype(np.float32))
    v = v.to(torch.bfloat16).reshape(B * n, Hk, d)
    pair.prefill(0, list(range(B)), [n] * B, k.reshape(B * n, Hk, d), v, torch.ones((B * n, Hk)), 0.5)
    q = torch.zeros((B, G * Hk, d), dtype=torch.bfloat16)
    q[:, :, 0] = 1
    out, ref = pair.attend(0, list(range(B)), q, 1.0)
    assert np.isfinite(ref).all() and np.abs(ref).max() > 4e37
    # 2^-16 of the largest value for the weights, and a few parts in a million for the exponentials
    assert np.isfinite(out).all() and np.abs(out - ref).max() <= 2 * (2.0 ** -16 + 1e-5) * 1e38, np.abs(out - ref).max()
