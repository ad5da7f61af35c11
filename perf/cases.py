"""The work that a user of this library has it do, as measurable cases.

A case is a dict of plain values; `kind` says which part of a program it stands for:

  prompt  whole requests through one attention layer: chunk attention and admission of ragged prompts
          (scores given, or from the linear write gate), decode steps, the slots freed at the end
  decode  one new token of a running batch through several layers: promotion of all layers ahead, then per
          layer the ring write and the ragged paged attention
  select  the same with read-time page selection: landmark upkeep, page scoring, attention over the picked pages
  admit   admission of long prompts into the paged dual cache, the slots freed at the end
  mlp     the Write-Gate MLP over the keys of a chunk
  evict   a prompt under a memory budget: admission, eviction scores, removal, attention over what is left
  train   training-time Write-Gated Attention of packed sequences: forward, sparsity term, backward

Model shapes are those of wgkv_workloads (32 query / 8 kv heads of 128, bf16; 8 / 2 heads of 64, fp32) and the other
head shapes that a pool accepts.  Sequence lengths and admission rates follow from the case alone, so that inputs of
two seeds cost the same; the values come from the seed.
"""
import math
import random

import numpy as np
import torch

import paper_2512_17452_amd as wg

TAU = 0.5
DEV = "cuda:0"
DECODE_ROOM = 8192  # tokens that a decode case's slots can grow by
TOKENS = 64         # new tokens that a decode case's inputs hold; a pass takes the next one


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def _heads(hq=32, hk=8, d=128, dtype="bf16"):
    return {"hq": hq, "hk": hk, "d": d, "dtype": dtype}


def listed():
    return [
        # the smallest request: the tiny workload (fp32, 512-token prompt, 16 decode steps), where launches count
        {"name": "request_tiny_f32", "kind": "prompt", **_heads(8, 2, 64, "f32"), "w": 64, "page": 16, "batch": 1,
         "len_min": 512, "len_max": 512, "chunk": 512, "steps": 16, "hidden": 0, "rates": "uniform"},
        # a batch of short chat-size requests of odd lengths
        {"name": "request_short_b8", "kind": "prompt", **_heads(), "w": 256, "page": 16, "batch": 8,
         "len_min": 131, "len_max": 1501, "chunk": 1024, "steps": 8, "hidden": 0, "rates": "beta_2_8"},
        # one user decoding at 32K context through a 32-layer model
        {"name": "decode_b1_32k", "kind": "decode", **_heads(), "w": 256, "page": 16, "batch": 1, "layers": 32,
         "len_min": 32768, "len_max": 32768, "rates": "beta_2_8"},
        # the benchmark's decode step: batch 8, contexts of 64K to 128K
        {"name": "decode_b8_128k", "kind": "decode", **_heads(), "w": 256, "page": 16, "batch": 8, "layers": 8,
         "len_min": 65537, "len_max": 131072, "rates": "beta_1p5_8"},
        # the large ragged batch: 32 sequences, heads from nearly empty to nearly dense
        {"name": "decode_b32_64k_ragged", "kind": "decode", **_heads(), "w": 128, "page": 32, "batch": 32, "layers": 4,
         "len_min": 65536, "len_max": 65536, "rates": "ragged_mix"},
        # decode with page selection at 2048 keys per head
        {"name": "select_b8_128k", "kind": "select", **_heads(), "w": 256, "page": 16, "batch": 8, "layers": 4,
         "len_min": 65537, "len_max": 131072, "rates": "beta_1p5_8", "budget": 128},
        # chunked prefill of long prompts with the linear gate on a 4096-wide hidden state
        {"name": "prefill_16k_b2", "kind": "prompt", **_heads(), "w": 256, "page": 16, "batch": 2,
         "len_min": 14001, "len_max": 16384, "chunk": 4096, "steps": 0, "hidden": 4096, "rates": "half"},
        # the same for a model of 64-wide heads
        {"name": "prefill_6k_d64", "kind": "prompt", **_heads(32, 8, 64), "w": 256, "page": 16, "batch": 1,
         "len_min": 6001, "len_max": 6001, "chunk": 2048, "steps": 0, "hidden": 2048, "rates": "half"},
        # admission alone of a 100K-token prompt whose scores are known
        {"name": "admit_100k", "kind": "admit", **_heads(), "w": 256, "page": 16, "batch": 1,
         "len_min": 100003, "len_max": 100003, "rates": "beta_1p5_8"},
        # the write gate of one 4 x 4096-token chunk
        {"name": "gate_mlp_16k", "kind": "mlp", **_heads(), "tokens": 16384, "width": 512},
        # eviction rounds of 64 heads at about 4.5K entries with 256 observation queries
        {"name": "evict_b8_18k", "kind": "evict", **_heads(), "w": 256, "page": 16, "batch": 8,
         "len_min": 18001, "len_max": 18001, "rates": "quarter", "obs": 256},
        # one training sample of 16K tokens
        {"name": "train_16k", "kind": "train", **_heads(), "w": 256, "seqs": 1, "len_min": 16384, "len_max": 16384},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_TUNED = _heads()
_OTHERS = [_heads(32, 8, 64), _heads(64, 8, 128), _heads(16, 8, 128), _heads(8, 8, 128), _heads(8, 2, 64, "f32"),
           _heads(16, 4, 128, "f32")]


def _draw_heads(rng):
    return dict(_TUNED if rng.random() < 0.6 else rng.choice(_OTHERS))


def draw(rng):
    kind = rng.choice(["prompt", "prompt", "prompt", "decode", "decode", "select", "admit", "mlp", "evict", "train"])
    page, w = rng.choice([16, 16, 16, 32, 64]), rng.choice([64, 100, 128, 256, 256, 512])
    rates = rng.choice(["uniform", "beta_2_8", "beta_1p5_8", "ragged_mix"])
    c = {"kind": kind}
    if kind == "prompt":
        c.update(_draw_heads(rng))
        tuned = {k: c[k] for k in _TUNED} == _TUNED
        batch = rng.choice([1, 1, 2, 3, 5, 8])
        hi = max(200, _log_int(rng, 200, 16384 if tuned else 5000) // max(1, batch if not tuned else batch // 2))
        lo = rng.randint(max(1, hi // 8), hi)
        gate = rng.random() < 0.4 and c["hk"] <= 16 and c["dtype"] == "bf16"
        c.update(w=w, page=page, batch=batch, len_min=lo, len_max=hi, chunk=rng.choice([512, 1000, 2048, 4096]),
                 steps=rng.choice([0, 0, 1, 4, 16]), hidden=rng.choice([1024, 2048, 4096]) if gate else 0,
                 rates="half" if gate else rates)
    elif kind in ("decode", "select"):
        c.update(_draw_heads(rng))
        batch = rng.choice([1, 2, 3, 4, 8, 16])
        layers = 16 if batch <= 2 else 8 if batch <= 4 else 4
        hi = _log_int(rng, 16384, 131072 if batch <= 8 else 65536)
        c.update(w=w, page=page, batch=batch, layers=layers, len_min=rng.randint(hi // 2, hi), len_max=hi,
                 rates="beta_1p5_8" if rates == "uniform" else rates)
        if kind == "select":
            c["budget"] = max(1, 2048 // page)
    elif kind == "admit":
        c.update(_draw_heads(rng))
        batch = rng.choice([1, 1, 2, 4])
        hi = _log_int(rng, 1000, 100000 // batch)
        c.update(w=w, page=page, batch=batch, len_min=rng.randint(max(1, hi // 4), hi), len_max=hi, rates=rates)
    elif kind == "mlp":
        c.update(_draw_heads(rng))
        c.update(tokens=_log_int(rng, 1, 16384 if c["dtype"] == "bf16" else 2048),
                 width=rng.choice([128, 256, 512, 512, 768, 200]))
        if c["width"] % 32:
            c["tokens"] = min(c["tokens"], 2048)
    elif kind == "evict":
        c.update(_draw_heads(rng))
        batch = rng.choice([1, 2, 4, 8])
        hi = _log_int(rng, 2000, 18000 if {k: c[k] for k in _TUNED} == _TUNED else 8000)
        c.update(w=w, page=page, batch=batch, len_min=rng.randint(hi // 2, hi), len_max=hi, rates=rates,
                 obs=rng.choice([32, 64, 256, 256]))
    else:
        seqs = rng.choice([1, 1, 2, 4, 7])
        hi = max(64, _log_int(rng, 300, 15000) // max(1, seqs // 2))
        c.update(_heads(*rng.choice([(32, 8), (32, 8), (16, 4)])))
        c.update(w=w, seqs=seqs, len_min=rng.randint(max(1, hi // 3), hi), len_max=hi)
    return c


# ---------------------------------------------------------------------------------------------
# what follows from a case alone
# ---------------------------------------------------------------------------------------------
def _lens(c, n):
    """n lengths spread evenly over [len_min, len_max], in a shuffled order."""
    lo, hi = c["len_min"], c["len_max"]
    out = [lo + (hi - lo) * i // max(1, n - 1) for i in range(n)] if n > 1 else [hi]
    random.Random(n).shuffle(out)
    return out


def _rates(c, layers):
    """Admission rate of every (layer, kv head)."""
    r = np.random.RandomState(7)
    shape = (layers, c["hk"])
    law = c["rates"]
    if law == "uniform":
        out = r.uniform(0.10, 0.40, shape)
    elif law == "beta_2_8":
        out = r.beta(2.0, 8.0, shape)
    elif law == "beta_1p5_8":
        out = r.beta(1.5, 8.0, shape)
    elif law == "quarter":
        out = np.full(shape, 0.25)
    elif law == "half":
        out = np.full(shape, 0.5)
    else:  # 5 % of the heads nearly dense, 20 % nearly empty, the rest so that the mean is 0.10
        u = (r.permutation(shape[0] * shape[1]) + 0.5).reshape(shape) / (shape[0] * shape[1])
        out = np.full(shape, (0.10 - 0.05 * 0.9 - 0.20 * 0.01) / 0.75)
        out[u < 0.05] = 0.9
        out[(u >= 0.05) & (u < 0.25)] = 0.01
    return np.clip(out, 0.005, 0.95)


def _dt(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _es(c):
    return 4 if c["dtype"] == "f32" else 2


def _gen(seed, *key):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(np.random.SeedSequence([int(seed), *[int(k) for k in key]]).generate_state(1, dtype=np.uint64)[0] >> 1))
    return g


def _normal(c, gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=_dt(c))


def _scores(gen, n, rates):
    """Scores [n, heads] that pass TAU at the given rates."""
    u = torch.rand((n, len(rates)), generator=gen, device=DEV, dtype=torch.float64)
    b = torch.as_tensor(math.log(1.0 - TAU) / np.log(rates), device=DEV)
    return (1.0 - torch.pow(1.0 - u, b)).clamp_(0.0, 1.0).to(torch.float32).contiguous()


def _pool(c, layers, slots, max_len, n_pages, call_seqs, call_tokens):
    cfg = wg.Config(layers, c["hq"], c["hk"], c["d"], wg.F32 if c["dtype"] == "f32" else wg.BF16, c["page"], c["w"],
                    slots, -(-max_len // c["page"]) + 2, int(n_pages))
    return wg.Pool(cfg, call_seqs, call_tokens)


def _attend64(q, k, v, see):
    """softmax(q k^T / sqrt(d)) v in 64 bits for the queries q [n, G, d] of one kv head; see [n, keys] or None."""
    n, G, d = q.shape
    s = torch.matmul(q.double().reshape(n * G, d), k.double().t()) / math.sqrt(d)
    if see is not None:
        s.view(n, G, -1).masked_fill_(~see[:, None, :], float("-inf"))
    s -= s.amax(dim=1, keepdim=True)
    s.exp_()
    out = torch.matmul(s, v.double()) / s.sum(dim=1, keepdim=True)
    return out.view(n, G, d)


# ---------------------------------------------------------------------------------------------
# prompt
# ---------------------------------------------------------------------------------------------
def _prompt_inputs(c, seed):
    """Per chunk step: (slots, token counts, q, k, v, scores or None, hidden or None); then the decode tokens."""
    rates = _rates(c, 1)[0]
    lens, done, steps = _lens(c, c["batch"]), [0] * c["batch"], []
    gate_w = None
    if c["hidden"]:
        gate_w = (0.02 * torch.randn((c["hk"], c["hidden"]), generator=_gen(seed, 9), device=DEV)).to(_dt(c))
    while any(d < n for d, n in zip(done, lens)):
        ids = [s for s in range(c["batch"]) if done[s] < lens[s]]
        nt = [min(c["chunk"], lens[s] - done[s]) for s in ids]
        gen, tot = _gen(seed, 1, len(steps)), sum(nt)
        q, k, v = (_normal(c, gen, tot, h, c["d"]) for h in (c["hq"], c["hk"], c["hk"]))
        hidden = _normal(c, gen, tot, c["hidden"]) if c["hidden"] else None
        g = None if c["hidden"] else _scores(gen, tot, rates)
        steps.append((ids, nt, q, k, v, g, hidden))
        for s, n in zip(ids, nt):
            done[s] += n
    gen = _gen(seed, 2)
    B = c["batch"]
    dec = [tuple(_normal(c, gen, B, h, c["d"]) for h in (c["hq"], c["hk"], c["hk"])) + (_scores(gen, B, rates),)
           for _ in range(c["steps"])]
    return steps, dec, gate_w


def _prepare_prompt(c, seed):
    steps, dec, gate_w = _prompt_inputs(c, seed)
    B, lens = c["batch"], _lens(c, c["batch"])
    n_pages = sum((-(-(n + c["steps"]) // c["page"]) + 2 + -(-c["w"] // c["page"])) * c["hk"] for n in lens)
    pool = _pool(c, 1, B, max(lens) + c["steps"], n_pages, B, max(sum(s[1]) for s in steps))
    outs = [torch.empty((sum(s[1]), c["hq"], c["d"]), dtype=torch.float32, device=DEV) for s in steps]
    dec_out = torch.empty((max(1, len(dec)), B, c["hq"], c["d"]), dtype=torch.float32, device=DEV)
    return {"pool": pool, "steps": steps, "dec": dec, "gate_w": gate_w, "outs": outs, "dec_out": dec_out,
            "dec_rows": list(dec_out.unbind(0)), "ids": list(range(B)), "scale": 1.0 / math.sqrt(c["d"])}


def _run_prompt(st):
    pool, scale = st["pool"], st["scale"]
    for (ids, nt, q, k, v, g, hidden), out in zip(st["steps"], st["outs"]):
        if g is None:
            g = wg.gate_scores(hidden, st["gate_w"])
        pool.attend(0, ids, q, out, scale, n_q=nt, k_chunk=k, v_chunk=v, g_chunk=g, tau=TAU)
        pool.prefill_admit(0, ids, nt, k, v, g, tau=TAU)
    for (q, k, v, g), out in zip(st["dec"], st["dec_rows"]):
        pool.decode_step(0, st["ids"], k, v, g, tau=TAU)
        pool.attend(0, st["ids"], q, out, scale)
    for s in st["ids"]:
        pool.free_seq(s)
    res = {"prefill": st["outs"]}
    if st["dec"]:
        res["decode"] = st["dec_out"]
    return res


def _exact_prompt(c, seed):
    steps, dec, gate_w = _prompt_inputs(c, seed)
    B, G, W = c["batch"], c["hq"] // c["hk"], c["w"]
    hist = [[] for _ in range(B)]
    outs = [torch.zeros((sum(s[1]), c["hq"], c["d"]), dtype=torch.float64, device=DEV) for s in steps]
    where = [[] for _ in range(B)]
    for i, (ids, nt, q, k, v, g, hidden) in enumerate(steps):
        if g is None:
            g = torch.sigmoid(hidden.double() @ gate_w.double().t())
        base = 0
        for s, n in zip(ids, nt):
            hist[s].append((q[base:base + n], k[base:base + n], v[base:base + n], g[base:base + n].double()))
            where[s].append((i, base, n))
            base += n
    dec_out = torch.zeros((max(1, len(dec)), B, c["hq"], c["d"]), dtype=torch.float64, device=DEV)
    for s in range(B):
        n_prompt = sum(n for _, _, n in where[s])
        q, k, v, g = (torch.cat([h[x] for h in hist[s]] + [t[x][s:s + 1].to(hist[s][0][x].dtype) for t in dec])
                      for x in range(4))
        pos = torch.arange(q.shape[0], device=DEV)
        rows = max(1, int(2.5e8) // (G * q.shape[0]))
        for h in range(c["hk"]):
            for i0 in range(0, q.shape[0], rows):
                i = pos[i0:i0 + rows]
                e = int(i[-1]) + 1
                see = (pos[None, :e] <= i[:, None]) & ((i[:, None] - pos[None, :e] < W) | (g[None, :e, h] >= TAU))
                o = _attend64(q[i0:i0 + rows, h * G:(h + 1) * G], k[:e, h], v[:e, h], see)
                at = 0
                for step, base, n in where[s]:  # this sequence's positions [at, at + n) are rows base.. of that step
                    lo, hi = max(i0, at), min(i0 + len(i), at + n)
                    if lo < hi:
                        outs[step][base + lo - at:base + hi - at, h * G:(h + 1) * G] = o[lo - i0:hi - i0]
                    at += n
                for t in range(len(dec)):
                    if i0 <= n_prompt + t < i0 + len(i):
                        dec_out[t, s, h * G:(h + 1) * G] = o[n_prompt + t - i0]
    res = {"prefill": outs}
    if dec:
        res["decode"] = dec_out
    return res


def _visible(n, w, rate):
    """Pairs (query, visible key) of one sequence and head, expected."""
    m = min(n, w)
    return m * (m + 1) / 2 + (n - m) * w + rate * (n - m) * (n - m + 1) / 2


def _work_prompt(c):
    rates, lens, es = _rates(c, 1)[0], _lens(c, c["batch"]), _es(c)
    G, flops, nbytes = c["hq"] // c["hk"], 0.0, 0.0
    for n in lens:
        t = n + c["steps"]
        flops += sum(4.0 * c["d"] * G * _visible(t, c["w"], r) for r in rates)
        nbytes += t * (c["hq"] * c["d"] * (es + 4) + c["hk"] * (2 * c["d"] * es + 4))          # q, out, k, v, scores
        nbytes += sum(min(t, c["w"]) + r * max(0, t - c["w"]) for r in rates) * 2 * c["d"] * es  # rows written
        nbytes += c["steps"] * sum(min(n, c["w"]) + r * max(0, n - c["w"]) for r in rates) * 2 * c["d"] * es
        nbytes += n * c["hidden"] * es
        flops += 2.0 * n * c["hidden"] * c["hk"]
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------------------------
# decode, select
# ---------------------------------------------------------------------------------------------
def _history(c, seed, layer, s, n, rates):
    gen = _gen(seed, 3, layer, s)
    k, v = (_normal(c, gen, n, c["hk"], c["d"]) for _ in range(2))
    return k, v, _scores(gen, n, rates[layer])


def _new_tokens(c, seed, rates):
    gen = _gen(seed, 4)
    L, B = c["layers"], c["batch"]
    q, k, v = (_normal(c, gen, TOKENS, L, B, h, c["d"]) for h in (c["hq"], c["hk"], c["hk"]))
    g = torch.stack([_scores(gen, TOKENS * B, rates[layer]).view(TOKENS, B, c["hk"]) for layer in range(L)], dim=1)
    return q, k, v, g.contiguous()


def _prepare_decode(c, seed):
    L, B, lens, rates = c["layers"], c["batch"], _lens(c, c["batch"]), _rates(c, c["layers"])
    P, nlp = c["page"], -(-c["w"] // c["page"])
    # the pages of the admitted entries, of one prompt's worst case at a time while it is admitted, and of the new tokens
    pages = sum(math.ceil(1.1 * r * n / P) + 64 + nlp + DECODE_ROOM // P for n in lens for r in rates.ravel())
    pages += c["hk"] * (max(lens) // P + 2)
    pool = _pool(c, L, B, max(lens) + DECODE_ROOM, pages, B, max(lens))
    for layer in range(L):
        for s, n in enumerate(lens):
            k, v, g = _history(c, seed, layer, s, n, rates)
            pool.prefill_admit(layer, [s], [n], k, v, g, tau=TAU)
            pool.status()
    toks = _new_tokens(c, seed, rates)
    toks = [[[x[t, layer] for x in toks] for layer in range(L)] for t in range(TOKENS)]
    out = torch.empty((L, B, c["hq"], c["d"]), dtype=torch.float32, device=DEV)
    st = {"pool": pool, "toks": toks, "out": out, "rows": list(out.unbind(0)), "ids": list(range(B)), "at": 0,
          "scale": 1.0 / math.sqrt(c["d"])}
    if c["kind"] == "select":
        st["landmarks"] = pool.quest_landmarks()
        st["stride"] = -(-(max(lens) + DECODE_ROOM) // P)
        st["scores"] = [torch.zeros((B * c["hk"], st["stride"]), dtype=torch.float32, device=DEV) for _ in range(L)]
        st["budget"] = c["budget"]
        for layer in range(L):
            pool.quest_update(layer, st["ids"], st["landmarks"], reset=True)
    return st


def _run_decode(st):
    pool, ids, scale, toks = st["pool"], st["ids"], st["scale"], st["toks"][st["at"] % TOKENS]
    st["at"] += 1
    pool.decode_promote(ids, tau=TAU)
    for layer, ((q, k, v, g), out) in enumerate(zip(toks, st["rows"])):
        pool.decode_step(layer, ids, k, v, g, tau=TAU)
        pool.attend(layer, ids, q, out, scale)
    return st["out"]


def _run_select(st):
    pool, ids, scale, toks = st["pool"], st["ids"], st["scale"], st["toks"][st["at"] % TOKENS]
    st["at"] += 1
    pool.decode_promote(ids, tau=TAU)
    picked = []
    for layer, ((q, k, v, g), out) in enumerate(zip(toks, st["rows"])):
        pool.decode_step(layer, ids, k, v, g, tau=TAU)
        pool.quest_update(layer, ids, st["landmarks"])
        _, sel, cnt = pool.quest_select(layer, ids, q, st["landmarks"], st["budget"], st["stride"],
                                        scores=st["scores"][layer])
        pool.attend_selected(layer, ids, q, sel, cnt, out, scale)
        picked += [sel, cnt]
    return {"out": st["out"], "picked": picked, "scores": st["scores"]}


def _exact_decode(c, seed):
    L, B, lens, rates = c["layers"], c["batch"], _lens(c, c["batch"]), _rates(c, c["layers"])
    G, W, P = c["hq"] // c["hk"], c["w"], c["page"]
    qn, kn, vn, _ = _new_tokens(c, seed, rates)
    out = torch.zeros((L, B, c["hq"], c["d"]), dtype=torch.float64, device=DEV)
    stride = -(-(max(lens) + DECODE_ROOM) // P)
    scores = [torch.zeros((B * c["hk"], stride), dtype=torch.float64, device=DEV) for _ in range(L)]
    for layer in range(L):
        for s, n in enumerate(lens):
            k, v, g = _history(c, seed, layer, s, n, rates)
            first = max(0, n + 1 - W)  # the new token is position n: the window holds [n + 1 - W, n]
            for h in range(c["hk"]):
                old = torch.nonzero(g[:first, h] >= TAU).view(-1)
                q = qn[0, layer, s, h * G:(h + 1) * G].double()
                if c["kind"] == "select" and len(old):
                    ko = k[old, h].double()
                    pad = -(-len(old) // P) * P - len(old)  # the last page repeats its last entry
                    pages = torch.cat([ko, ko[-1:].expand(pad, -1)]).view(-1, P, c["d"])
                    lo, hi = pages.amin(1), pages.amax(1)
                    u = torch.maximum(q[:, None] * lo[None], q[:, None] * hi[None]).sum(2).amax(0)
                    scores[layer][s * c["hk"] + h, :len(u)] = u
                    if len(u) > c["budget"]:
                        keep = torch.zeros(len(u), dtype=torch.bool, device=DEV)
                        keep[torch.sort(u, descending=True, stable=True).indices[:c["budget"]]] = True
                        old = old[keep.repeat_interleave(P)[:len(old)]]
                kk = torch.cat([k[old, h], k[first:, h], kn[0, layer, s, h][None]])
                vv = torch.cat([v[old, h], v[first:, h], vn[0, layer, s, h][None]])
                out[layer, s, h * G:(h + 1) * G] = _attend64(q[None], kk, vv, None)[0]
    if c["kind"] == "select":
        return {"out": out, "picked": [None] * (2 * L), "scores": scores}
    return out


def _work_decode(c):
    es, nbytes, flops = _es(c), 0.0, 0.0
    for n in _lens(c, c["batch"]):
        for r in _rates(c, c["layers"]).ravel():
            old = r * max(0, n - c["w"])
            read = old
            if c["kind"] == "select":
                read = min(old, c["budget"] * c["page"])
                nbytes += old / c["page"] * (2 * c["d"] * es + 4)
            keys = read + min(n, c["w"])
            nbytes += keys * 2 * c["d"] * es + c["hq"] // c["hk"] * c["d"] * (es + 4) + 2 * c["d"] * es * (2 + r)
            flops += 4.0 * c["d"] * c["hq"] / c["hk"] * keys
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------------------------
# admit
# ---------------------------------------------------------------------------------------------
def _admit_inputs(c, seed):
    lens, gen = _lens(c, c["batch"]), _gen(seed, 5)
    k, v = (_normal(c, gen, sum(lens), c["hk"], c["d"]) for _ in range(2))
    return lens, k, v, _scores(gen, sum(lens), _rates(c, 1)[0])


def _prepare_admit(c, seed):
    lens, k, v, g = _admit_inputs(c, seed)
    # a pool for the admitted cache: the caller's bound on what a head admits keeps the host's accounting there
    bound = int(max(lens) * min(1.0, 1.1 * _rates(c, 1).max()) + 64)
    n_pages = len(lens) * c["hk"] * (-(-bound // c["page"]) + 1 + -(-c["w"] // c["page"]))
    pool = _pool(c, 1, len(lens), max(lens), n_pages, len(lens), sum(lens))
    mask = torch.zeros((sum(lens), c["hk"]), dtype=torch.uint8, device=DEV)
    return {"pool": pool, "ids": list(range(len(lens))), "lens": lens, "k": k, "v": v, "g": g, "mask": mask,
            "bound": bound, "pages": pool.pool_pages(), "free": pool.meta()["free_stack"]}


def _run_admit(st):
    pool = st["pool"]
    pool.prefill_admit(0, st["ids"], st["lens"], st["k"], st["v"], st["g"], tau=TAU, admit_mask_out=st["mask"],
                       max_admitted_per_head=st["bound"])
    for s in st["ids"]:
        pool.free_seq(s)
    # the rows stay in the pool's pages and the order of the pages in the free list, so both say what was written where
    return {"mask": st["mask"], "pages": st["pages"], "free": st["free"]}


def _work_admit(c):
    es, nbytes = _es(c), 0.0
    for n in _lens(c, c["batch"]):
        rows = sum(r * max(0, n - c["w"]) + min(n, c["w"]) for r in _rates(c, 1)[0])
        nbytes += n * c["hk"] * 5 + rows * 4 * c["d"] * es
    return {"bytes": nbytes, "flops": 0.0}


# ---------------------------------------------------------------------------------------------
# mlp
# ---------------------------------------------------------------------------------------------
def _prepare_mlp(c, seed):
    gen, T, H, d, n = _gen(seed, 6), c["tokens"], c["hk"], c["d"], c["width"]
    k, kr = 1.5 * _normal(c, gen, T, H, d), 0.7 * _normal(c, gen, T, H, d)
    w1 = (torch.randn((H, n, 2 * d), generator=gen, device=DEV) * (2 * d) ** -0.5).to(_dt(c))
    b1 = 0.5 * torch.randn((H, n), generator=gen, device=DEV)
    w2 = (torch.randn((H, n), generator=gen, device=DEV) * 2.0 * n ** -0.5).to(_dt(c))
    b2 = torch.randn((H,), generator=gen, device=DEV)
    return {"args": (k, kr, w1, b1, w2, b2), "out": torch.empty((T, H), dtype=torch.float32, device=DEV)}


def _run_mlp(st):
    return wg.gate_mlp_scores(*st["args"], out=st["out"])


def _exact_mlp(c, seed):
    k, kr, w1, b1, w2, b2 = (x.double() for x in _prepare_mlp(c, seed)["args"])
    x = torch.cat([y / torch.sqrt((y * y).mean(-1, keepdim=True) + 1e-6) for y in (k, kr)], dim=-1)
    if c["dtype"] == "bf16":
        x = x.to(torch.bfloat16).double()  # the features enter the first product in the model's type
    out = torch.empty(x.shape[:2], dtype=torch.float64, device=DEV)
    for h in range(c["hk"]):
        z = torch.nn.functional.gelu(x[:, h].contiguous() @ w1[h].t() + b1[h])
        out[:, h] = torch.sigmoid(z @ w2[h] + b2[h])
    return out


def _work_mlp(c):
    es, T, H, d, n = _es(c), c["tokens"], c["hk"], c["d"], c["width"]
    return {"bytes": T * H * (2 * d * es + 4) + H * n * (2 * d * es + es + 4), "flops": T * H * (4.0 * d * n + 2 * n)}


# ---------------------------------------------------------------------------------------------
# evict
# ---------------------------------------------------------------------------------------------
def _prepare_evict(c, seed):
    lens, k, v, g = _admit_inputs(c, seed)
    B = len(lens)
    bound = int(max(lens) * min(1.0, 1.1 * _rates(c, 1).max()) + 64)
    n_pages = B * c["hk"] * (-(-bound // c["page"]) + 1 + -(-c["w"] // c["page"]))
    pool = _pool(c, 1, B, max(lens), n_pages, B, sum(lens))
    gen = _gen(seed, 7)
    q_obs, q = _normal(c, gen, B, c["obs"], c["hq"], c["d"]), _normal(c, gen, B, c["hq"], c["d"])
    return {"pool": pool, "ids": list(range(B)), "lens": lens, "k": k, "v": v, "g": g, "bound": bound, "q_obs": q_obs,
            "q": q, "out": torch.empty((B, c["hq"], c["d"]), dtype=torch.float32, device=DEV),
            "gone": torch.zeros((B * c["hk"],), dtype=torch.int32, device=DEV), "scale": 1.0 / math.sqrt(c["d"])}


def _run_evict(st):
    pool, ids = st["pool"], st["ids"]
    pool.prefill_admit(0, ids, st["lens"], st["k"], st["v"], st["g"], tau=TAU, max_admitted_per_head=st["bound"])
    raw, scores = pool.evict_scores(0, ids, st["q_obs"], st["scale"], st["bound"])
    pool.evict_apply(0, ids, scores, 0.1, n_evicted_out=st["gone"])
    pool.attend(0, ids, st["q"], st["out"], st["scale"])
    for s in ids:
        pool.free_seq(s)
    return {"raw": raw, "scores": scores, "gone": st["gone"], "out": st["out"]}


def _exact_evict(c, seed):
    lens, k, v, g = _admit_inputs(c, seed)
    B, G, W, H = len(lens), c["hq"] // c["hk"], c["w"], c["hk"]
    bound = int(max(lens) * min(1.0, 1.1 * _rates(c, 1).max()) + 64)
    gen = _gen(seed, 7)
    q_obs, q = _normal(c, gen, B, c["obs"], c["hq"], c["d"]), _normal(c, gen, B, c["hq"], c["d"])
    raw, scores = (torch.zeros((B * H, bound), dtype=torch.float64, device=DEV) for _ in range(2))
    out, base = torch.zeros((B, c["hq"], c["d"]), dtype=torch.float64, device=DEV), 0
    for b, n in enumerate(lens):
        for h in range(H):
            kh, vh, gh = k[base:base + n, h].double(), v[base:base + n, h].double(), g[base:base + n, h]
            old = torch.nonzero(gh[:max(0, n - W)] >= TAU).view(-1)
            if len(old):
                qo = q_obs[b, :, h * G:(h + 1) * G].double().reshape(-1, c["d"])
                a = torch.softmax(torch.matmul(qo, kh[old].t()) / math.sqrt(c["d"]), dim=1)
                s = a.view(c["obs"], G, -1).amax(1).sum(0)
                p = torch.nn.functional.max_pool1d(s[None, None], 5, stride=1, padding=2)[0, 0]
                raw[b * H + h, :len(old)], scores[b * H + h, :len(old)] = s, p
                drop = math.floor(float(np.float32(0.1)) * len(old))
                # pooling makes runs of equal scores, and among equal ones the older goes first; in 32 bits they are equal too
                keep = torch.sort(torch.sort(p.float(), stable=True).indices[drop:]).values
                old = old[keep]
            at = torch.cat([old, torch.arange(max(0, n - W), n, device=DEV)])
            out[b, h * G:(h + 1) * G] = _attend64(q[b, h * G:(h + 1) * G][None], kh[at], vh[at], None)[0]
        base += n
    return {"raw": raw, "scores": scores, "gone": None, "out": out}


def _work_evict(c):
    w = _work_admit(c)
    es, G = _es(c), c["hq"] // c["hk"]
    entries = sum(r * max(0, n - c["w"]) for n in _lens(c, c["batch"]) for r in _rates(c, 1)[0])
    rows = c["batch"] * c["hq"] * c["obs"]
    # keys for the scores, rows that move up (nearly all behind the first removed one), what the attention reads
    w["bytes"] += entries * (c["d"] * es + 8) + rows * c["d"] * es + 0.9 * entries * 6 * c["d"] * es
    w["flops"] += 2.0 * c["d"] * c["obs"] * G * entries + 4.0 * c["d"] * G * 0.9 * entries
    return w


# ---------------------------------------------------------------------------------------------
# train
# ---------------------------------------------------------------------------------------------
def _prepare_train(c, seed):
    lens, gen = _lens(c, c["seqs"]), _gen(seed, 8)
    rows = sum(lens)
    q, k, v = (_normal(c, gen, rows, h, c["d"]) for h in (c["hq"], c["hk"], c["hk"]))
    g = torch.rand((rows, c["hk"]), generator=gen, device=DEV)
    dout = _normal(c, gen, rows, c["hq"], c["d"])
    return {"lens": lens, "q": q, "k": k, "v": v, "g": g, "dout": dout, "w": c["w"], "scale": 1.0 / math.sqrt(c["d"])}


def _run_train(st):
    a = (st["q"], st["k"], st["v"], st["g"])
    out, lse = wg.soft_attn_forward(*a, st["lens"], st["w"], st["scale"], 1e-6)
    loss, dg_loss = wg.sparsity_loss(st["g"])
    dq, dk, dv, dg = wg.soft_attn_backward(*a, out, lse, st["dout"], st["lens"], st["w"], st["scale"], 1e-6)
    return {"out": out, "lse": lse, "loss": loss, "dg_loss": dg_loss, "dq": dq, "dk": dk, "dv": dv, "dg": dg}


def _exact_train(c, seed):
    st = _prepare_train(c, seed)
    G, W, scale, eps, base = c["hq"] // c["hk"], c["w"], st["scale"], 1e-6, 0
    g = st["g"].double()
    res = {n: torch.zeros(st[s].shape, dtype=torch.float64, device=DEV)
           for n, s in (("out", "q"), ("dq", "q"), ("dk", "k"), ("dv", "v"), ("dg", "g"))}
    res["lse"] = torch.zeros((len(g), c["hq"]), dtype=torch.float64, device=DEV)
    for n in st["lens"]:
        pos = torch.arange(n, device=DEV)
        for h in range(c["hk"]):
            kh, vh, gh = (x[base:base + n, h].double().contiguous() for x in (st["k"], st["v"], g))
            rows = max(1, int(1.5e8) // n)
            for i0 in range(0, n, rows):
                i = pos[i0:i0 + rows]
                e = int(i[-1]) + 1
                near = i[:, None] - pos[None, :e] < W
                one = gh.new_ones(())
                m = torch.where(near, torch.maximum(one, gh[None, :e]), gh[None, :e])
                bias = (m + eps).log_().masked_fill_(pos[None, :e] > i[:, None], float("-inf"))
                follows = (~near) & (gh[None, :e] > 0)
                at = slice(base + i0, base + i0 + len(i))
                for qh in range(h * G, (h + 1) * G):
                    q, do = st["q"][at, qh].double(), st["dout"][at, qh].double()
                    s = torch.matmul(q, kh[:e].t()).mul_(scale).add_(bias)
                    lse = torch.logsumexp(s, dim=1)
                    p = s.sub_(lse[:, None]).exp_()
                    o = torch.matmul(p, vh[:e])
                    res["out"][at, qh], res["lse"][at, qh] = o, lse
                    res["dv"][base:base + e, h] += torch.matmul(p.t(), do)
                    ds = torch.matmul(do, vh[:e].t()).sub_((do * o).sum(1, keepdim=True)).mul_(p)
                    res["dq"][at, qh] = torch.matmul(ds, kh[:e]) * scale
                    res["dk"][base:base + e, h] += torch.matmul(ds.t(), q) * scale
                    res["dg"][base:base + e, h] += ds.mul_(follows).sum(0) / (gh[:e] + eps)
        base += n
    res["loss"] = (g + g * (1 - g)).mean().view(1)
    res["dg_loss"] = (2 - 2 * g) / g.numel()
    return res


def _work_train(c):
    lens = _lens(c, c["seqs"])
    rows = sum(lens)
    nbytes = rows * (c["hq"] * c["d"] * (2 * 2 + 2 * 4) + c["hk"] * c["d"] * (2 * 2 + 2 * 4) + c["hk"] * 12 + c["hq"] * 4)
    return {"bytes": nbytes, "flops": sum(14.0 * c["d"] * c["hq"] * n * (n + 1) / 2 for n in lens)}


# ---------------------------------------------------------------------------------------------
_KINDS = {
    "prompt": (_prepare_prompt, _run_prompt, _exact_prompt, _work_prompt),
    "decode": (_prepare_decode, _run_decode, _exact_decode, _work_decode),
    "select": (_prepare_decode, _run_select, _exact_decode, _work_decode),
    "admit": (_prepare_admit, _run_admit, lambda c, seed: None, _work_admit),
    "mlp": (_prepare_mlp, _run_mlp, _exact_mlp, _work_mlp),
    "evict": (_prepare_evict, _run_evict, _exact_evict, _work_evict),
    "train": (_prepare_train, _run_train, _exact_train, _work_train),
}


def prepare(case, seed):
    st = _KINDS[case["kind"]][0](case, seed)
    st["kind"] = case["kind"]
    return st


def run(state):
    return _KINDS[state["kind"]][1](state)


def exact(case, seed):
    return _KINDS[case["kind"]][2](case, seed)


def work(case):
    return _KINDS[case["kind"]][3](case)


def tolerance(case):
    """About four times the error against 64 bits that the paths show."""
    if case["kind"] == "admit":
        return "exact"  # rows are copied and pages handed out in a fixed order
    if case["kind"] == "mlp":
        return {"rel": 3e-5}  # features that land on the other side of a bf16 rounding boundary
    wide = {k: case[k] for k in _TUNED} == _TUNED or case["kind"] == "train"
    # the 128-wide, four-heads-a-group bf16 kernels round the softmax weights to bf16; the others keep 32 bits.
    # An eviction or a page selection whose cut falls between two nearly equal scores may take the other of the two.
    rel = 7e-3 if wide or case["kind"] in ("evict", "select") else 5e-6
    return {"rel": rel, "differ": 0.01 if case["kind"] == "select" else 0.0}
