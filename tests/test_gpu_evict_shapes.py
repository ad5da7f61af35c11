"""Eviction scores on the matrix cores for every bf16 head shape: caches that end on and around a wave's 16 rows, a tile of 64 and of
128 keys and a block's keys, windows of 32 query rows and more that fill a tile or end inside it, pages that hold a wave's
rows and pages that do not, and the three ways of sharing keys between waves."""
import math

import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G", [(d, G) for d in (64, 128) for G in (1, 2, 4, 8)])
@pytest.mark.parametrize("P,Hk,rows,lens,scale", [
    (16, 1, 32, [1, 63], 1.0), (8, 2, 96, [64, 65, 15], -1.0), (64, 2, 160, [127, 129, 256], 1.0), (16, 2, 128, [255, 17], 0.0),
    (32, 49, 32, [200, 256], 1.0),            # two waves over the same keys
    (16, 86, 64, [64, 200, 192], 1.0),        # one
])
def test_scores_of_every_shape_match_fp64(d, G, P, Hk, rows, lens, scale):
    W, B, n_obs, dev = 16, len(lens), rows // G, torch.device("cuda:0")
    Hq, n_tok = G * Hk, [n + W for n in lens]     # everything behind the window is admitted
    max_gp, nlp = max(n_tok) // P + 2, -(-W // P)
    pool = wg.Pool(wg.Config(1, Hq, Hk, d, wg.BF16, P, W, B, max_gp, B * Hk * (max_gp + nlp) + 8), B, sum(n_tok))
    gen = torch.Generator().manual_seed(d + G + rows)
    k, v = (torch.randn((sum(n_tok), Hk, d), generator=gen).bfloat16() for _ in range(2))
    q = torch.randn((B, n_obs, Hq, d), generator=gen).bfloat16()
    g = torch.ones((sum(n_tok), Hk))
    pool.prefill_admit(0, list(range(B)), n_tok, k.to(dev), v.to(dev), g.to(dev), tau=0.5)
    sc = scale / math.sqrt(d)
    raw, pooled = pool.evict_scores(0, list(range(B)), q.to(dev), sc, max(lens) + 3)
    assert pool.status()[1] == 0
    raw, pooled = raw.cpu().numpy(), pooled.cpu().numpy()
    base = 0
    for s, n in enumerate(lens):
        for h in range(0, Hk, max(1, Hk // 7)):
            K = k[base:base + n, h].double().numpy()
            x = q[s, :, h * G:(h + 1) * G].double().numpy() @ K.T * sc            # [n_obs, G, n]
            p = np.exp(x - x.max(-1, keepdims=True))
            ref = (p / p.sum(-1, keepdims=True)).max(1).sum(0)
            # fp32 sums of hardware exponentials (an ulp each), scores exact to about d * 2^-24 * |s|
            np.testing.assert_allclose(raw[s * Hk + h, :n], ref, rtol=1e-5, atol=0)
            pad = np.pad(raw[s * Hk + h, :n], 2, constant_values=-np.inf)
            np.testing.assert_array_equal(pooled[s * Hk + h, :n], np.lib.stride_tricks.sliding_window_view(pad, 5).max(-1))
            assert not raw[s * Hk + h, n:].any() and not pooled[s * Hk + h, n:].any()
        base += n_tok[s]
