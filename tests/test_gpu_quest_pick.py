"""Which pages are picked, against a stable sort of the scores the call returns: caches from one page to more than the threads of a
block hold in registers, numbers of pages around what a thread owns, a budget of one, of nearly all and of more than there are, runs
of equal scores at the cut."""
import numpy as np
import pytest
import torch

import paper_2512_17452_amd as wg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("distinct", [10 ** 6, 7], ids=["scores", "ties"])
@pytest.mark.parametrize("lens,budget", [([1, 2, 255, 256, 257, 300], 100), ([512, 513, 1023, 1025, 4095, 4097], 128), ([5200, 4200, 900], 899),
                                         ([700, 64, 5000], 1), ([40, 3, 1], 50)])
def test_picks_of_a_stable_sort(lens, budget, distinct):
    W, d, B = 1, 64, len(lens)
    pool = wg.Pool(wg.Config(1, 2, 2, d, wg.BF16, 1, W, B, max(lens) + 2, sum(2 * (n + 3) for n in lens)), B, sum(lens) + B)
    rng = np.random.default_rng(sum(lens) + budget)
    ids, nt = list(range(B)), [n + 1 for n in lens]  # the last token stays in the ring
    k = rng.standard_normal((sum(nt), 2, d)).astype(np.float32)
    if distinct < 10:  # keys from a handful of rows: pages of equal scores
        k = k[rng.integers(0, distinct, sum(nt))]
    k = torch.from_numpy(k).to(torch.bfloat16).cuda()
    pool.prefill_admit(0, ids, nt, k, k, torch.ones((sum(nt), 2), device="cuda"), tau=0.5)
    lm = pool.quest_landmarks()
    pool.quest_update(0, ids, lm, reset=True)
    q = torch.from_numpy(rng.standard_normal((B, 2, d)).astype(np.float32)).to(torch.bfloat16).cuda()
    scores, sel, cnt = pool.quest_select(0, ids, q, lm, budget, max(lens) + 5)
    scores, sel, cnt = scores.cpu().numpy(), sel.cpu().numpy(), cnt.cpu().numpy()
    for u in range(2 * B):
        n = lens[u // 2]
        want = np.sort(np.argsort(-scores[u, :n], kind="stable")[:min(n, budget)])
        assert cnt[u] == len(want)
        np.testing.assert_array_equal(sel[u, :len(want)], want)
        assert (sel[u, len(want):] == -1).all()


def test_empty_caches_with_rows_of_no_scores():
    """Every head's cache is empty and a score row has no elements: nothing is read from it, nothing picked."""
    B, d = 3, 64
    pool = wg.Pool(wg.Config(1, 2, 2, d, wg.BF16, 16, 32, B, 4, 60), B, 60)
    k = torch.randn((B, 2, d), device="cuda").to(torch.bfloat16)
    pool.prefill_admit(0, list(range(B)), [1] * B, k, k, torch.ones((B, 2), device="cuda"), tau=0.5)
    lm = pool.quest_landmarks()
    pool.quest_update(0, list(range(B)), lm, reset=True)
    room = torch.full((8,), float("nan"), device="cuda")  # the row would begin at its end
    sel = torch.full((2 * B, 5), 7, dtype=torch.int32, device="cuda")
    cnt = torch.full((2 * B,), 7, dtype=torch.int32, device="cuda")
    rc = pool.L.wgkv_quest_select(pool.h, 0, B, wg.binding._ids(range(B)), k.data_ptr(), lm.data_ptr(), lm.numel(), 5, room.data_ptr() + 32, 0,
                                  sel.data_ptr(), cnt.data_ptr(), wg.binding._stream())
    assert rc == 0 and (sel == -1).all() and (cnt == 0).all() and torch.isnan(room).all()
