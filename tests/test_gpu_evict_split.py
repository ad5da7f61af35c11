"""Eviction scores of the matrix-core path where its sweeps split the work differently: four, two or one waves over the same
keys by the number of 256-key blocks in the call (at most 96 and at most 256), caches that end on and around a tile of
64 and 128 keys, windows that end inside a tile of 64 query rows, and a negative and a zero scale."""
import math

import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hk,n_obs,lens,scale", [
    (1, 1, 8, [1], 1.0), (1, 2, 24, [63], 1.0), (2, 2, 40, [64, 65], -1.0), (2, 1, 16, [127, 129], 0.0),
    (4, 24, 8, [128, 256, 255, 1], 1.0),      # 96 blocks
    (2, 49, 8, [200, 256], 1.0),              # 98
    (2, 64, 24, [385, 300], 1.0),             # 256
    (3, 86, 8, [64, 200, 192], 1.0),          # 258
])
def test_scores_match_fp64(B, Hk, n_obs, lens, scale):
    d, P, W, G, dev = 128, 16, 16, 4, torch.device("cuda:0")
    Hq, n_tok = G * Hk, [n + W for n in lens]     # everything behind the window is admitted
    max_gp = max(n_tok) // P + 2
    pool = wg.Pool(wg.Config(1, Hq, Hk, d, wg.BF16, P, W, B, max_gp, B * Hk * (max_gp + 1) + 8), B, sum(n_tok))
    gen = torch.Generator().manual_seed(B + Hk + n_obs)
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
        for h in range(Hk):
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


def test_scores_of_queries_that_are_not_16_byte_aligned():
    """The matrix-core sweeps read queries 16 bytes at a time: others go to the general kernels, any element's address will do."""
    B, Hk, n_obs, n, d, W, dev = 2, 2, 16, 150, 128, 16, torch.device("cuda:0")
    pool = wg.Pool(wg.Config(1, 4 * Hk, Hk, d, wg.BF16, 16, W, B, 16, B * Hk * 18), B, B * (n + W))
    gen = torch.Generator(device=dev).manual_seed(4)
    k, v = (torch.randn((B * (n + W), Hk, d), generator=gen, device=dev).bfloat16() for _ in range(2))
    pool.prefill_admit(0, [0, 1], [n + W] * B, k, v, torch.ones((B * (n + W), Hk), device=dev), tau=0.5)
    q = torch.randn((B, n_obs, 4 * Hk, d), generator=gen, device=dev).bfloat16()
    room = torch.zeros(q.numel() + 8, dtype=torch.bfloat16, device=dev)
    raw, pooled = pool.evict_scores(0, [0, 1], q, 1 / math.sqrt(d), n)
    for off in (1, 2, 4):
        q_off = room[off:off + q.numel()].view(q.shape)
        q_off.copy_(q)
        assert q_off.data_ptr() % 16 != 0
        raw2, pooled2 = pool.evict_scores(0, [0, 1], q_off, 1 / math.sqrt(d), n)
        # both within 1e-5 of the definition (see above)
        torch.testing.assert_close(raw2, raw, rtol=2e-5, atol=0)
        torch.testing.assert_close(pooled2, pooled, rtol=2e-5, atol=0)
