"""Decode attention of bf16 pools at the edges of its pairs of tiles: one tile, an odd number of them, a last row anywhere in a
pair, more pairs than a wave keeps in LDS, more than 64 tiles of a region; pages that a freed slot left full of infinities; scales
of either sign and of zero.  Weights keep 16 bits and more here, so the tolerance is 2^-16 of the largest value and the fp32 sums."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_q, rand_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G", [(128, 4), (128, 1), (128, 8), (64, 4), (64, 2)])
@pytest.mark.parametrize("P", [2, 16, 64])
def test_pairs_of_tiles(d, G, P):
    rng = np.random.default_rng(d + G + P)
    lens, Hk, W = [1, 15, 16, 17, 31, 32, 33, 49, 129, 700, 2500], 2, 48
    B, max_gp = len(lens), 2500 // P + 2
    pages = (B + 1) * Hk * (max_gp + -(-W // P))
    pair = Pair(1, G * Hk, Hk, d, wg.BF16, P, W, B + 1, max_gp, pages, max_call_seqs=B, max_call_tokens=sum(lens))
    # the pages that are handed out next hold infinities
    n = 2500
    bad = torch.full((n, Hk, d), float("inf"), dtype=torch.bfloat16, device=pair.dev)
    pair.pool.prefill_admit(0, [B], [n], bad, bad, torch.ones((n, Hk), device=pair.dev), tau=0.5)
    pair.pool.free_seq(B)
    k, v, g = rand_tokens(rng, sum(lens), Hk, d, torch.bfloat16, rates=[0.6, 0.97])
    pair.orc.push_tokens(0, [B], [n], np.zeros((n, Hk, d), np.float32), np.zeros((n, Hk, d), np.float32), np.ones((n, Hk), np.float32), 0.5)
    pair.orc.free_seq(B)
    pair.prefill(0, list(range(B)), lens, k, v, g, 0.5)
    q = rand_q(rng, B, G * Hk, d, torch.bfloat16)
    for scale in (d ** -0.5, -d ** -0.5, 4 * d ** -0.5, 0.0):
        out, ref = pair.attend(0, list(range(B)), q, scale)
        # 2^-16 of the largest value for the weights; a score is off by some 1e-6 of it (fp32 sums of d products)
        tol = 2 * (2.0 ** -16 + 1e-6 * abs(scale) * d) * np.abs(v.float().numpy()).max()
        assert np.isfinite(out).all() and np.abs(out - ref).max() <= tol, (scale, np.abs(out - ref).max(), tol)
