"""The Write-Gate MLP at widths that are no multiple of the 32 hidden units of a chunk, in every form of the bf16 kernel, and the
fp32 kernel of 16-token blocks: sizes around the line at which it takes over, a last block and a last slice that are not full,
odd head dimensions.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg
from oracle import gate_mlp
from test_gpu_gate_mlp import _inputs

pytestmark = pytest.mark.gpu


def _check(dtype, T, Hk, d, width):
    ins = _inputs(dtype, T, Hk, d, width, T + width)
    g = wg.gate_mlp_scores(*[x.cuda() for x in ins], eps=1e-6).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(T, 70)), np.arange(max(0, T - 100), T), np.arange(0, T, 37)]))
    f = lambda x: x.float().numpy()
    _, ref = gate_mlp(f(ins[0])[rows], f(ins[1])[rows], *[f(x) for x in ins[2:]], eps=1e-6, feature_bf16=dtype == torch.bfloat16)
    return np.abs(g[rows] - ref)


@pytest.mark.parametrize("T,Hk,d,width", [(5, 2, 128, 1), (40, 8, 64, 33), (1024, 8, 128, 200), (1100, 8, 64, 95), (3000, 8, 128, 40),
                                          (5000, 8, 64, 200), (12500, 8, 128, 70), (13000, 8, 64, 31)])
def test_bf16_widths(T, Hk, d, width):
    err = _check(torch.bfloat16, T, Hk, d, width)
    # sums within 2e-5; a feature on the other side of a rounding boundary moves a score as derived for the other widths, with
    # fewer units weighing more: standard deviation of the logit's slope at most 2 * 0.67 * max(1, sqrt(32 / width)) / sqrt(2 d)
    step = 4 * 2 * 0.67 * max(1.0, (32 / width) ** 0.5) / (2 * d) ** 0.5 * 2.0 ** -6 / 4
    assert np.isfinite(err).all() and err.max() <= step and (err > 2e-5).mean() <= 1e-2, (err.max(), step)


@pytest.mark.parametrize("T,Hk,d,width", [(384, 2, 64, 512), (385, 2, 64, 512), (1001, 1, 128, 100), (769, 1, 40, 65), (300, 3, 33, 64),
                                          (500, 2, 160, 30)])
def test_fp32(T, Hk, d, width):
    err = _check(torch.float32, T, Hk, d, width)
    assert np.isfinite(err).all() and err.max() <= 2e-5, err.max()


@pytest.mark.parametrize("T,Hk,d,width", [(32, 8, 128, 97), (33, 8, 128, 97), (128, 2, 64, 1023), (129, 2, 64, 1023), (1, 1, 64, 99), (256, 1, 128, 500)])
def test_few_tokens_at_ragged_widths(T, Hk, d, width):
    """As many (token, head) pairs as stay with the plain kernel and a few more: the same order of a row's squares on both sides, so no
    more than the sums differ and a feature that they move across a rounding boundary."""
    err = _check(torch.bfloat16, T, Hk, d, width)
    step = 4 * 2 * 0.67 * max(1.0, (32 / width) ** 0.5) / (2 * d) ** 0.5 * 2.0 ** -6 / 4
    assert np.isfinite(err).all() and err.max() <= step and (err > 2e-5).mean() <= 1e-2, (err.max(), step)


@pytest.mark.parametrize("pairs,d,width", [(640, 128, 260), (1088, 64, 70), (1600, 64, 40), (2304, 64, 9), (1600, 16, 300), (1024, 32, 256), (1408, 20, 65),
                                           (1088, 40, 65), (1088, 128, 100), (2304, 160, 30)])
def test_fp32_lines(pairs, d, width):
    """As many (token, head) pairs as stay with the plain kernel, and one token more in blocks of 16."""
    for T in (pairs, pairs + 1):
        err = _check(torch.float32, T, 1, d, width)
        assert np.isfinite(err).all() and err.max() <= 2e-5, (T, err.max())
