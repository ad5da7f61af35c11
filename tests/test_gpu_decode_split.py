"""Decode attention at the edges of how a call is cut over the blocks: one token, units shorter than the smallest piece,
a unit of several pieces, more units than a wave has lanes, more units than the launch has blocks (even shares that
straddle units), sequences with nothing cached among them, pages smaller and larger than a tile; every head shape."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_q, rand_tokens

pytestmark = pytest.mark.gpu

SHAPES = [(dt, d, G) for dt in (wg.F32, wg.BF16) for d in (64, 128) for G in (1, 2, 4, 8)]
IDS = [f"{'f32' if dt == wg.F32 else 'bf16'}-d{d}-G{G}" for dt, d, G in SHAPES]


@pytest.mark.parametrize("dtype,d,G", SHAPES, ids=IDS)
@pytest.mark.parametrize("Hk,P,W,lens", [(1, 16, 64, [1, 0, 17]),
                                         (2, 32, 40, [2600, 41, 900]),                       # several pieces
                                         (2, 4, 33, [350, 1500]),                            # pages smaller than a tile
                                         (8, 16, 24, [1 + 7 * i % 90 for i in range(12)]),   # 96 units
                                         (8, 64, 20, [3 + 11 * i % 80 for i in range(34)])], # 272 units: even shares
                         ids=["one", "pieces", "page4", "units96", "units272"])
def test_every_cut_against_the_oracle(dtype, d, G, Hk, P, W, lens):
    rng = np.random.default_rng(d + 7 * G + len(lens))
    tdt = torch.float32 if dtype == wg.F32 else torch.bfloat16
    B, max_gp = len(lens), max(lens) // P + 2
    pair = Pair(1, G * Hk, Hk, d, dtype, P, W, B, max_gp, B * Hk * (max_gp + -(-W // P)) + 8, max_call_seqs=B,
                max_call_tokens=sum(lens))
    k, v, g = rand_tokens(rng, sum(lens), Hk, d, tdt, rates=list(np.linspace(0.3, 0.95, Hk)))
    pair.prefill(0, list(range(B)), lens, k, v, g, 0.5)
    order = list(rng.permutation(B))
    q = rand_q(rng, B, G * Hk, d, tdt)
    a, ref = pair.attend(0, order, q)
    b, _ = pair.attend(0, order, q)
    np.testing.assert_array_equal(a, b)  # counters are back at zero, the order of the sums is fixed
    # bf16, 128 wide, four heads a group: weights rounded to bf16; every other shape sums fp32 products
    tol = 1e-2 if (dtype, d, G) == (wg.BF16, 128, 4) else 2e-5
    assert np.isfinite(a).all() and np.abs(a - ref).max() <= tol, np.abs(a - ref).max()
