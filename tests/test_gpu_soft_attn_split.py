"""Training-time attention where the dK/dV kernel splits a kv head's work differently: four, two or one waves over the
same keys by the longest sequence (four only from 400 tokens on) and the number of 128-key blocks in the call.  Many short
sequences reach each form at sizes that the fp64 oracle checks whole; bars as in test_gpu_soft_attn.py."""
import math

import pytest
import torch

import paper_2512_17452_amd as wg
from test_gpu_soft_attn import BWD_MAX, BWD_MEAN, FWD_MAX, FWD_MEAN, LSE_TOL, _check, _inputs, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,n_seqs,longest,Hk,W", [
    (21, 16, 128, 8, 20),   # 128 blocks
    (22, 17, 128, 8, 20),   # 136
    (23, 64, 65, 8, 33),    # 512
    (24, 65, 65, 8, 33),    # 520
    (25, 43, 161, 8, 1),    # 688, two blocks of keys per sequence, ends inside a tile
    (26, 1, 399, 8, 40),    # 32 blocks, two waves per key group
    (27, 2, 400, 8, 40),    # 64: four
    (28, 3, 401, 4, 300),   # 48: four, heads that do not divide over the XCDs
    (29, 3, 401, 8, 40),    # 96: two
    (30, 24, 128, 8, 20),   # 192: the last of two at this length
    (31, 25, 128, 8, 20),   # 200: the first of one
    (32, 24, 200, 8, 20),   # 384: the last of two
    (33, 25, 200, 8, 20),   # 400: the first of one
    (34, 16, 97, 3, 20),    # three heads, sequences dealt over the XCDs
    (35, 7, 97, 5, 20),     # five heads dealt over them
])
def test_every_split_matches_fp64(seed, n_seqs, longest, Hk, W):
    n_tokens = [longest - (7 * i) % longest for i in range(n_seqs)]
    rows, scale = sum(n_tokens), 1 / math.sqrt(128)
    print("case", seed, n_seqs, longest, Hk, W, flush=True)
    q, k, v, g, dout = _inputs(seed, rows, Hk, "ends")
    qd, kd, vd, gd, dd = (x.to("cuda:0") for x in (q, k, v, g, dout))
    out, lse = wg.soft_attn_forward(qd, kd, vd, gd, n_tokens, W, scale, 1e-6)
    grads = wg.soft_attn_backward(qd, kd, vd, gd, out, lse, dd, n_tokens, W, scale, 1e-6)
    again = wg.soft_attn_backward(qd, kd, vd, gd, out, lse, dd, n_tokens, W, scale, 1e-6)
    torch.cuda.synchronize()
    ref_out, ref_lse, ref = _oracle(q, k, v, g, dout, n_tokens, W, scale, 1e-6)
    _check("out", out, ref_out, FWD_MAX, FWD_MEAN, False)
    _check("lse", lse, ref_lse, LSE_TOL, LSE_TOL, False)
    for name, got, rep, want in zip(("dq", "dk", "dv", "dg"), grads, again, ref):
        _check(name, got, want, BWD_MAX, BWD_MEAN, True)
        assert torch.equal(got, rep), name
