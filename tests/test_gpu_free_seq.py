"""wgkv_free_seq where its launch has several blocks: more pages than a block takes per turn, more (layer, kv head)
units than a block has threads, and slots that are freed without ever having been used.  State bit for bit against
the oracle, then the pages are handed out again."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from harness import Pair, rand_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers,Hk,P,W,T", [(1, 8, 1, 64, 900),     # 7.2K pages: eight blocks
                                               (40, 8, 16, 64, 90),    # 320 units: two windows of the prefix
                                               (33, 8, 4, 5, 70),      # a window of units that ends one unit long
                                               (2, 2, 16, 300, 40)])   # ring pages only, one block
def test_free_seq_in_several_blocks(n_layers, Hk, P, W, T):
    rng = np.random.default_rng(n_layers * 100 + T)
    tdt = torch.bfloat16
    max_gp = T // P + 4
    pair = Pair(n_layers, 4 * Hk, Hk, 64, wg.BF16, P, W, 3, max_gp, 2 * n_layers * Hk * (max_gp + -(-W // P)) + 8,
                max_call_seqs=2, max_call_tokens=2 * T, payload=False)
    rates = list(np.linspace(0.1, 0.95, Hk))
    for turn in range(2):
        for layer in range(n_layers):
            if layer == n_layers - 1 and n_layers > 1 and turn == 0:
                continue  # a layer of the slot that was never used
            lens = [T, max(1, T - 7 - layer)]
            k, v, g = rand_tokens(rng, sum(lens), Hk, 64, tdt, rates=rates)
            pair.prefill(layer, [0, 1], lens, k, v, g, 0.5)
        for s in (1, 2, 0):  # slot 2 holds nothing
            pair.pool.free_seq(s)
            pair.orc.free_seq(s)
            pair.check_state(payload=False)
