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


def _compare(pair, seqs, q, v_finite_max):
    out, ref = pair.attend(0, seqs, q, pair.cfg.head_dim ** -0.5)
    np.testing.assert_array_equal(np.isnan(out), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(out) * np.sign(out), np.isinf(ref) * np.sign(ref))
    ok = np.isfinite(ref)
    # 2^-16 of the largest value for the weights; a score is off by some 1e-6 of it
    assert np.abs(out[ok] - ref[ok]).max() <= 2 * (2.0 ** -16 + 1e-5) * v_finite_max
    return ~ok


# (lengths, kv heads): units of one piece and of several; more units than 64; ways of cutting where there are more units than blocks:
# whole units a wave, shares a wave, shares a block
CALLS = {"pieces": ([1, 17, 33, 250, 2500], 2), "shares": ([1, 17, 33, 250, 2500] * 5, 8), "solo": ([90] * 40, 8),
         "waves": ([40, 1100, 40, 200, 90, 40, 30, 60] * 5, 8), "blocks": ([1500] * 100 + [1, 17, 33, 250], 3)}


# the largest two in one shape of each path
CASES = [(c, d, G, 16) for c in CALLS for d, G in SHAPES if c not in ("shares", "blocks") or (d, G) in ((128, 4), (64, 1))] + \
    [(c, d, G, 4) for c in ("pieces", "solo") for d, G in SHAPES]


@pytest.mark.parametrize("call,d,G,P", CASES)
def test_what_is_not_finite_in_v_comes_out(call, d, G, P):
    """+inf, -inf, both and NaN in rows that are read: exactly the elements that they reach are not finite, as in a sum of weights
    times values."""
    lens, Hk = CALLS[call]
    rng = np.random.default_rng(d + G + len(lens))
    W, B = 16, len(lens)
    pages = sum(Hk * (n // P + 2 + -(-W // P)) for n in lens)
    pair = Pair(1, G * Hk, Hk, d, wg.BF16, P, W, B, max(lens) // P + 2, pages, max_call_seqs=B, max_call_tokens=sum(lens))
    k, v, _ = rand_tokens(rng, sum(lens), Hk, d, torch.bfloat16)
    top = float(v.float().abs().max())
    base = np.cumsum([0] + lens)
    inf = float("inf")
    for b, n in enumerate(lens):
        for h in range(Hk):
            if (b + h) % 7 == 6:
                continue  # a unit of finite values among them
            for col, vals in ((3, (inf,)), (17, (-inf,)), (40, (inf, -inf)), (41, (inf, inf, inf)), (63, (float("nan"),))):
                for x in vals[:n]:
                    row = int(rng.choice([0, n - 1, rng.integers(0, n)]))  # the oldest, the youngest (in the ring), any
                    v[base[b] + row, h, (col + 5 * b) % d] = x
    pair.prefill(0, list(range(B)), lens, k, v, torch.ones((sum(lens), Hk)), 0.5)
    bad = _compare(pair, list(range(B)), (0.3 * torch.from_numpy(rng.standard_normal((B, G * Hk, d)).astype(np.float32))).to(torch.bfloat16), top)
    assert bad.any() and not bad.all()


@pytest.mark.parametrize("d,G", [(128, 4), (64, 1), (64, 8)])
def test_infinities_far_below_the_largest_score(d, G):
    """Infinities under weights that are too small for fp32, in a tile, a wave, a block and a partial of their own: an infinity all the
    same, as in a sum of exact weights."""
    rng = np.random.default_rng(d * G)
    n, W, P, Hk = 3000, 16, 16, 2
    for gap in (80.0, 130.0, 300.0):  # powers of two under the largest weight
        for at in (0, 20, 100, 1500, 2990):
            pair = Pair(1, G * Hk, Hk, d, wg.BF16, P, W, 1, n // P + 2, 2 * Hk * (n // P + 3), max_call_seqs=1, max_call_tokens=n)
            k = torch.zeros((n, Hk, d), dtype=torch.bfloat16)
            k[:, :, 0] = gap * 0.6931
            k[at, :, 0] = 0
            _, v, _ = rand_tokens(rng, n, Hk, d, torch.bfloat16)
            v[at, :, 5], v[at, :, 6] = float("inf"), float("-inf")
            pair.prefill(0, [0], [n], k, v, torch.ones((n, Hk)), 0.5)
            q = torch.zeros((1, G * Hk, d), dtype=torch.bfloat16)
            q[:, :, 0] = 1
            out, ref = pair.attend(0, [0], q, 1.0)
            assert (ref[..., 5] == np.inf).all() and (ref[..., 6] == -np.inf).all() and np.isinf(ref).sum() == 2 * G * Hk
            np.testing.assert_array_equal(np.isfinite(out), np.isfinite(ref))
            np.testing.assert_array_equal(out[~np.isfinite(ref)], ref[~np.isfinite(ref)])
            ok = np.isfinite(ref)
            assert np.abs(out[ok] - ref[ok]).max() <= 1e-3


@pytest.mark.parametrize("d,G,B", [(128, 1, 16), (128, 1, 17), (64, 1, 16), (64, 1, 17), (64, 2, 32), (64, 2, 33), (128, 2, 33)])
def test_units_around_the_line_between_the_two_units(d, G, B):
    """Groups of few heads, as many units as go to the matrix cores and one more: the same sums."""
    rng = np.random.default_rng(d + G + B)
    lens, W, P = [1 + 37 * b % 900 for b in range(B)], 32, 16
    pair = Pair(1, G, 1, d, wg.BF16, P, W, B, 60, 70 * B, max_call_seqs=B, max_call_tokens=sum(lens))
    k, v, g = rand_tokens(rng, sum(lens), 1, d, torch.bfloat16)
    pair.prefill(0, list(range(B)), lens, k, v, g, 0.5)
    q = torch.from_numpy(rng.standard_normal((B, G, d)).astype(np.float32)).to(torch.bfloat16)
    out, ref = pair.attend(0, list(range(B)), q)
    assert np.isfinite(out).all() and np.abs(out - ref).max() <= 2 * (2.0 ** -16 + 1e-6 * d ** 0.5) * float(v.float().abs().max())
