"""The forms of the Write-Gate MLP kernel against the fp64 oracle: calls just inside and outside the sizes at which the
next form takes over, numbers of hidden-unit chunks that do not divide over the waves, and keys that are not finite."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from oracle import gate_mlp
from test_gpu_gate_mlp import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Hk,d,width", [(1, 1, 64, 32), (33, 3, 128, 96), (1024, 8, 64, 160),     # split, one round full
                                          (1025, 8, 128, 32), (4096, 8, 64, 96),                    # two unit groups
                                          (4097, 8, 128, 32), (12288, 8, 64, 32),                   # one group
                                          (12289, 8, 128, 64), (12700, 8, 64, 96),                  # two columns a wave
                                          # widths up to 64 are one group (two columns past the last line with 64)
                                          (1, 8, 128, 64), (12300, 8, 128, 32), (1024, 8, 128, 96), (1025, 8, 128, 96),
                                          (4097, 8, 64, 96), (12288, 8, 128, 96)])
def test_every_form_matches_fp64(T, Hk, d, width):
    ins = _inputs(torch.bfloat16, T, Hk, d, width, T + width)
    g = wg.gate_mlp_scores(*[x.cuda() for x in ins], eps=1e-6).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(T, 70)), np.arange(max(0, T - 300), T), np.arange(0, T, 37)]))
    f = lambda x: x.float().numpy()
    _, ref = gate_mlp(f(ins[0])[rows], f(ins[1])[rows], *[f(x) for x in ins[2:]], eps=1e-6, feature_bf16=True)
    err = np.abs(g[rows] - ref)
    # fp32 sums, GELU and sigmoid stay within 2e-5.  A feature whose fp32 normalisation lands on the other side of a
    # bf16 rounding boundary (a few in a million) moves by 2^-6 at |x| < 4, the logit by that times a sum over the units of
    # w2 gelu' w1, standard deviation 2 * 0.67 / sqrt(2 d) <= 0.12, and the score by a quarter of it: four of those.
    assert np.isfinite(g).all() and err.max() <= 4 * 0.12 * 2.0 ** -6 / 4 and (err > 2e-5).mean() <= 1e-2


@pytest.mark.parametrize("T", [40, 1500, 5000, 13000])
def test_a_key_that_is_not_finite_spoils_its_own_score_only(T):
    ins = _inputs(torch.bfloat16, T, 8, 128, 64, 3)
    clean = wg.gate_mlp_scores(*[x.cuda() for x in ins]).cpu()
    ins[0][T // 2, 3, 7] = float("nan")
    ins[1][T - 1, 0, 100] = float("inf")   # inf / inf in its norm
    g = wg.gate_mlp_scores(*[x.cuda() for x in ins]).cpu()
    bad = torch.zeros_like(g, dtype=torch.bool)
    bad[T // 2, 3] = bad[T - 1, 0] = True
    assert torch.isnan(g[bad]).all() and torch.equal(g[~bad], clean[~bad])
