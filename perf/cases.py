"""The work a program has this library do, as cases that can be timed and compared.

A case is one pass through the public entry points: a decode step over a few
attention layers of one model (``RetroLayer.step``, with the calls that go
around it), the same step as separate calls, a whole re-embedding stack
(``RetroDecoder.step``), or the prompt's storage (``retro_prefill_kv``).

* ``listed()``: the cases; ``draw(rng)``: one more of the same ranges.
* ``prepare(case, seed)``: the layers, their caches and the next inputs.
* ``run(state)``: one pass; calling it again decodes the next token.  After
  ``GEN`` tokens the sequences go back to the end of their prompts, as a program
  does that answers the next request on the same prompt.
* ``work(case)``, ``tolerance(case)``, ``exact(case, seed)``: the bytes and
  operations a pass cannot do without, how far another correct implementation
  may be off, and the outputs in 64 bits.

Several layers per pass keep each layer's cache out of the 256 MB last-level
cache between its own steps, as the other layers of a model do.
"""
from __future__ import annotations

import math

import torch

from paper_2508_09001_amd import binding as B
from paper_2508_09001_amd.decode import RetroDecoder
from paper_2508_09001_amd.layer import RetroLayer

GEN = 64      # tokens decoded after a prompt before the next request
INPUTS = 8    # distinct inputs, used in turn
T0 = 1020     # step number after the prompt (a multiple of every reuse interval drawn)

_TD = {"bf16": torch.bfloat16, "f32": torch.float32}

_BASE = dict(kind="step", batch=1, kv_heads=8, group=4, head_dim=128, page=16, budget=2048,
             permille=0, window=16, ctx=32768, ragged=False, tokens=1, update=False, reuse=0,
             outlier=False, dtype="bf16", layers=6, chunk=0)


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # the smallest layer that the tests and the benchmark know: launches and
        # hand-offs are all there is to it
        _case("step-2k-f32", kv_heads=2, head_dim=64, budget=256, window=4, ctx=2048, dtype="f32"),
        # one user on a Llama-3-8B-shaped model at 32K: the benchmark's headline layer
        _case("step-32k", outlier=True),
        # a serving batch of requests of mixed lengths
        _case("step-32k-b16", batch=16, budget=1024, window=8, ragged=True, layers=2),
        # long generations in the middle of their growth, eight tokens a step and a
        # wide window: 264 rows per KV head
        _case("step-32k-b4-w32", batch=4, group=8, budget=4096, window=32, tokens=8, layers=2),
        # the longest context with the widest window
        _case("step-131k-w64", page=32, budget=8192, window=64, ctx=131072, layers=4),
        # the same context with a budget that keeps every page: dense attention through
        # the retrospective path, the most a step can move
        _case("step-131k-dense", page=32, budget=132096, window=16, ctx=131072, layers=1),
        # the paper's efficiency setting: batch 8, a budget of 0.15 of the context, the
        # window's keys and values re-embedded before the step
        _case("step-32k-b8-rel", batch=8, permille=150, window=7, update=True, layers=2),
        # a program that puts work of its own between the parts of a step
        _case("split-64k-b4", kind="split", batch=4, budget=2048, window=8, ctx=65536, layers=2),
        # a prompt stored chunk by chunk, of a length that fills no chunk or page
        _case("prefill-30k", kind="prefill", ctx=30011, chunk=8192, layers=1, window=0),
        # the re-embedding stack of a Llama-shaped model, one user
        _case("decoder-32k-w16", kind="decoder", layers=4),
        # the same stack serving eight users: 72 rows through every projection
        _case("decoder-32k-b8-w8", kind="decoder", batch=8, window=8, layers=2),
        # a stack held in fp32
        _case("decoder-8k-f32", kind="decoder", budget=1024, window=4, ctx=8192, dtype="f32",
              layers=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: kinds by how often a program makes the
    call, sizes spread over their logarithms, odd lengths and groups among them."""
    top = [work(c) for c in listed()]
    most = {k: max(w[k] for w in top) for k in ("bytes", "flops")}
    while True:
        kind = rng.choice(["step"] * 5 + ["split"] + ["prefill"] + ["decoder"] * 2)
        c = dict(_BASE, kind=kind)
        c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        c["page"] = rng.choice([16, 16, 32])
        c["ctx"] = _log(rng, 1000, 131072)
        c["kv_heads"] = rng.choice([1, 2, 4, 5, 8, 8, 8])
        c["group"] = rng.choice([1, 2, 3, 4, 4, 4, 7, 8])
        c["head_dim"] = rng.choice([64, 128, 128])
        c["batch"] = rng.choice([1, 1, 2, 3, 4, 8, 13, 16])
        c["window"] = rng.choice([0, 1, 2, 4, 7, 8, 16, 16, 32, 64])
        c["ragged"] = c["batch"] > 1 and rng.random() < 0.6
        c["budget"] = min(_log(rng, 128, 16384), c["ctx"])
        if rng.random() < 0.2:
            c["permille"] = rng.choice([50, 100, 150, 250])
        c["outlier"] = rng.random() < 0.3
        c["layers"] = rng.choice([1, 2, 4, 6])
        if kind == "step":
            c["tokens"] = rng.choice([1] * 8 + [2, 8])
            c["update"] = c["window"] > 0 and rng.random() < 0.2
            c["reuse"] = rng.choice([0] * 9 + [2, 3])
        elif kind == "prefill":
            c.update(window=0, layers=1, permille=0,
                     chunk=rng.choice([0, 512, 2048, 8192, 1000]))
        elif kind == "decoder":
            # model widths of the tests' and the benchmark's stacks
            c["kv_heads"], c["group"], c["head_dim"] = rng.choice(
                [(8, 4, 128), (8, 4, 128), (4, 4, 64), (8, 4, 64), (4, 8, 128)])
            c["batch"] = rng.choice([1, 1, 2, 4, 8])
            c["window"] = rng.choice([0, 2, 4, 8, 16])
            c["ctx"] = min(c["ctx"], 65536)
            c["layers"] = rng.choice([1, 2, 4])
            if c["batch"] * (c["window"] + 1) > 112:
                continue
        w = work(c)
        if w["bytes"] > most["bytes"] or w["flops"] > most["flops"]:
            continue
        if c["budget"] < c["page"] or c["layers"] * c["batch"] * c["ctx"] > 1 << 21:
            continue
        if c["dtype"] == "f32" and c["batch"] * c["ctx"] > 1 << 18:
            continue
        return c


# ---- sizes -----------------------------------------------------------------------

def _lens(c):
    """Prompt lengths: all ctx, or spread over [ctx / 4, ctx]."""
    if not c["ragged"]:
        return [c["ctx"]] * c["batch"]
    return [int(c["ctx"] * (0.25 + 0.75 * ((0.618034 * (b + 1)) % 1.0))) for b in range(c["batch"])]


def _max_pages(c):
    """Table length: the longest prompt and room for the tokens to come."""
    return -(-(c["ctx"] + GEN * c["tokens"] + 256) // c["page"])


def _keep(c, length):
    """Pages a step keeps of a sequence of `length` tokens."""
    bt = max(c["budget"], length * c["permille"] // 1000)
    return min(bt // c["page"], -(-length // c["page"]))


def work(case):
    c = case
    elt = 2 if c["dtype"] == "bf16" else 4
    hk, hq, d, P, W, b = (c["kv_heads"], c["kv_heads"] * c["group"], c["head_dim"], c["page"],
                          c["window"], c["batch"])
    row = hk * d * elt
    if c["kind"] == "prefill":
        n = sum(_lens(c))
        pages = sum(-(-x // P) for x in _lens(c))
        return {"bytes": 4.0 * n * row + 2.0 * pages * row, "flops": 0.0}
    n_new = c["tokens"]
    lens = [x + n_new for x in _lens(c)]
    pages = sum(-(-x // P) for x in lens)
    kept = sum(_keep(c, x) for x in lens)
    toks = sum(min(_keep(c, x) * P, x) for x in lens)
    rows = W + 1
    nbytes = 2.0 * pages * row                         # page digests
    nbytes += 4.0 * pages * (hk + 1)                   # last-loaded steps, page table
    nbytes += 2.0 * toks * row                         # keys and values of the kept pages
    nbytes += b * rows * hq * d * elt                  # window queries
    nbytes += (2.0 * b * W + b * rows) * hq * (d + 1) * 4   # output cache, outputs
    nbytes += 12.0 * kept * hk + n_new * b * 8.0 * row
    if c["update"] or c["kind"] == "decoder":
        nbytes += b * W * 4.0 * row
    flops = 4.0 * pages * hq * d + 4.0 * toks * rows * hq * d
    if c["kind"] == "decoder":
        dm = hq * d
        wts = dm * (2 * dm + 2 * hk * d)
        nbytes += wts * elt + b * rows * dm * 12.0
        flops += 2.0 * wts * b * rows
    return {"bytes": nbytes * c["layers"], "flops": flops * c["layers"]}


# How far another correct implementation at the same precision may be off, about
# four times what the path shows against exact().  Selections, masks, lengths and
# stored keys are the same bit for bit: the score's fp32 order is part of the
# method's definition here.
def tolerance(case):
    if case["kind"] == "prefill":
        return "exact"
    if case["kind"] == "decoder":
        # bf16 stacks round between layers; a changed rounding of a query can exchange
        # pages of nearly equal score
        return {"rel": 4e-3, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-5, "max": 4e-4} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 1e-4}


# ---- inputs ----------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, shape, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)


def _prompt(c, g):
    """Keys and values of every sequence of one layer, [n][h_k][d]; with outliers,
    four channels of every KV head are eight times as large, as in trained keys."""
    hk, d, td = c["kv_heads"], c["head_dim"], _TD[c["dtype"]]
    scale = torch.ones(hk, d, device="cuda")
    if c["outlier"]:
        ch = torch.rand(hk, d, generator=g, device="cuda").topk(4, dim=1).indices
        scale.scatter_(1, ch, 8.0)
    out = []
    for n in _lens(c):
        k = torch.randn(n, hk, d, generator=g, device="cuda")
        k *= scale
        out.append((k.to(td), _randn(g, (n, hk, d), td)))
    return out, scale


def _layer_inputs(c, g):
    """One layer: the prompt, the next INPUTS steps' window queries and tokens, the
    window's state in the middle of a generation."""
    b, hk, G, d, W = c["batch"], c["kv_heads"], c["group"], c["head_dim"], c["window"]
    hq, td, mp = hk * G, _TD[c["dtype"]], _max_pages(c)
    prompt, scale = _prompt(c, g)
    x = dict(prompt=prompt, scale=scale)
    x["table"] = torch.randperm(b * mp, generator=g, device="cuda").to(torch.int32).view(b, mp)
    # every step's query: noise plus half of an earlier key, so that pages differ in score
    hist = torch.randn(b, INPUTS + W, hq, d, generator=g, device="cuda")
    for s, (k, _) in enumerate(prompt):
        r = torch.randint(0, k.shape[0], (INPUTS + W, hq), generator=g, device="cuda")
        hist[s] += 0.5 * k[r, torch.arange(hq, device="cuda") // G].float()
    hist = hist.to(td)
    x["q"] = [hist[:, i:i + W + 1].contiguous() for i in range(INPUTS)]
    shape = (c["tokens"], b, hk, d)
    x["k"] = [(torch.randn(shape, generator=g, device="cuda") * scale).to(td)
              for _ in range(INPUTS)]
    x["v"] = [_randn(g, shape, td) for _ in range(INPUTS)]
    if c["update"]:
        x["ku"] = [(torch.randn(b, W, hk, d, generator=g, device="cuda") * scale).to(td)
                   for _ in range(INPUTS)]
        x["vu"] = [_randn(g, (b, W, hk, d), td) for _ in range(INPUTS)]
    _window_state(c, g, x)
    return x


def _window_state(c, g, x):
    b, hk, W, mp = c["batch"], c["kv_heads"], c["window"], _max_pages(c)
    hq, d = hk * c["group"], c["head_dim"]
    ago = torch.randint(1, W + 9, (b, hk, mp), generator=g, device="cuda")
    seen = torch.rand(b, hk, mp, generator=g, device="cuda") < 0.25
    x["A"] = torch.where(seen, T0 - ago, torch.full_like(ago, -1)).to(torch.int32)
    x["oc"] = 0.05 * torch.randn(b, max(W, 1), hq, d, generator=g, device="cuda")
    base = 22.0 if c["outlier"] else math.log(c["budget"]) + 0.6
    x["zc"] = base + 0.3 * torch.randn(b, max(W, 1), hq, generator=g, device="cuda")


def _layer_args(c, table=None):
    return dict(batch=c["batch"], num_kv_heads=c["kv_heads"], group=c["group"],
                head_dim=c["head_dim"], page_size=c["page"], budget=c["budget"],
                window=c["window"], max_pages=_max_pages(c), dtype=c["dtype"],
                budget_permille=c["permille"], reuse_interval=c["reuse"], page_table=table)


def _resume(lay, x):
    lay.last_loaded.copy_(x["A"])
    lay.o_cache.copy_(x["oc"])
    lay.lse_cache.copy_(x["zc"])


def _stack_inputs(c, seed):
    """The weights, prompts and embeddings of a re-embedding stack."""
    g = _gen(seed)
    td, L = _TD[c["dtype"]], c["layers"]
    hq_d, hk_d = c["kv_heads"] * c["group"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    dm = hq_d

    def w(rows, cols, scale):
        return (torch.randn(rows, cols, generator=g, device="cuda") * scale).to(td)

    weights = [dict(wq=w(dm, hq_d, dm ** -0.5), wk=w(dm, hk_d, dm ** -0.5),
                    wv=w(dm, hk_d, dm ** -0.5), wo=w(hq_d, dm, (hq_d * L) ** -0.5))
               for _ in range(L)]
    per = []
    for _ in range(L):
        prompt, _scale = _prompt(dict(c, outlier=False), g)
        x = dict(prompt=prompt)
        _window_state(dict(c, outlier=False), g, x)
        per.append(x)
    emb = _randn(g, (c["batch"], INPUTS + c["window"], dm), td)
    wins = [emb[:, i:i + c["window"] + 1].contiguous() for i in range(INPUTS)]
    return weights, per, wins


def prepare(case, seed):
    c = case
    st = dict(case=c, i=0)
    if c["kind"] == "decoder":
        weights, per, wins = _stack_inputs(c, seed)
        kw = _layer_args(c)
        kw.pop("page_table")
        dec = RetroDecoder(weights, **kw)
        for n, x in enumerate(per):
            for s, (k, v) in enumerate(x["prompt"]):
                dec.prefill(n, s, k, v)
            _resume(dec.layers[n], x)
        dec.decoded = T0     # the window's tokens were decoded, not part of a prompt
        st.update(dec=dec, wins=wins, layers=dec.layers)
    else:
        g = _gen(seed)
        st["layers"], st["x"] = [], []
        for _ in range(c["layers"]):
            x = _layer_inputs(c, g)
            lay = RetroLayer(**_layer_args(c, x["table"]))
            if c["kind"] == "prefill":
                st["src"] = x["prompt"]
            else:
                for s, (k, v) in enumerate(x["prompt"]):
                    lay.prefill(s, k, v)
                _resume(lay, x)
            st["layers"].append(lay)
            st["x"].append({n: x[n] for n in ("q", "k", "v", "ku", "vu") if n in x})
    st["lens"] = [lay.seq_lens.clone() for lay in st["layers"]]
    st["A"] = [lay.last_loaded.clone() for lay in st["layers"]]
    return st


def run(state):
    c, i = state["case"], state["i"]
    if c["kind"] == "prefill":
        return _run_prefill(state)
    if i == GEN:     # the next request on the same prompt
        i = state["i"] = 0
        for lay, n, a in zip(state["layers"], state["lens"], state["A"]):
            lay.seq_lens.copy_(n)
            lay.last_loaded.copy_(a)
    t = T0 + i
    state["i"] += 1
    if c["kind"] == "decoder":
        h = state["dec"].step(t, state["wins"][i % INPUTS])
        return {"h": h, "lse": [lay.lse_out for lay in state["layers"]],
                "lens": [lay.seq_lens for lay in state["layers"]]}
    j = i % INPUTS
    for lay, x in zip(state["layers"], state["x"]):
        q, k, v = x["q"][j], x["k"][j], x["v"][j]
        if c["update"]:
            lay.update_kv(x["ku"][j], x["vu"][j])
        if c["tokens"] > 1:
            lay.append_tokens(t, k[:-1], v[:-1])
        if c["kind"] == "split":
            lay.append(t, k[-1], v[-1])
            lay.select(t, q[:, c["window"]])
            lay.attend(t, q)
            lay.merge(t)
        else:
            lay.step(t, q, k[-1], v[-1])
    return [{"o": lay.o_out, "lse": lay.lse_out, "selected": lay.selected, "mask": lay.mask,
             "num_selected": lay.num_selected, "o_cache": lay.o_cache, "lse_cache": lay.lse_cache,
             "last_loaded": lay.last_loaded, "lens": lay.seq_lens} for lay in state["layers"]]


def _run_prefill(state):
    """New prompts stored over the sequences' old ones."""
    c, lay = state["case"], state["layers"][0]
    lay.seq_lens.zero_()
    for s, (k, v) in enumerate(state["src"]):
        n = k.shape[0]
        chunk = c["chunk"] or n
        for at in range(0, n, chunk):
            m = min(chunk, n - at)
            B.retro_prefill_kv(lay.dims, lay.cache, s, at, m, k[at:at + m], v[at:at + m])
    return {"k": lay.k_cache, "v": lay.v_cache, "digest": lay.digest, "lens": lay.seq_lens}


# ---- the outputs in 64 bits --------------------------------------------------------

def _digests(keys, P):
    """Element-wise minimum and maximum of every page's stored keys [n][h_k][d]:
    two [h_k][pages][d] in fp32 (exact: they are stored values)."""
    n, hk, d = keys.shape
    pad = -n % P
    k = keys.float()
    lo = torch.cat([k, k.new_full((pad, hk, d), math.inf)]).view(-1, P, hk, d).amin(1)
    hi = torch.cat([k, k.new_full((pad, hk, d), -math.inf)]).view(-1, P, hk, d).amax(1)
    return lo.transpose(0, 1), hi.transpose(0, 1)


def _scores(q, lo, hi):
    """Page scores [h_k][pages] for q [h_k][G][d], in the fp32 order that defines the
    selection: rounded products, a binary tree over d, the heads in order."""
    total = None
    for gq in range(q.shape[1]):
        qg = q[:, gq].float()[:, None]
        x = torch.maximum(qg * lo, qg * hi)
        while x.shape[-1] > 1:
            x = x[..., 0::2] + x[..., 1::2]
        total = x[..., 0] if total is None else total + x[..., 0]
    return total + 0.0


def _exact_step(c, t, q, keys, vals, n_new, A, oc, zc, k_max):
    """One step of one layer in 64 bits.  q [b][W+1][h_q][d]; keys / vals: per
    sequence [n][h_k][d] with the step's n_new tokens; A, oc, zc as before the step."""
    b, hk, G, d, P, W = (c["batch"], c["kv_heads"], c["group"], c["head_dim"], c["page"],
                         c["window"])
    hq = hk * G
    dev = q.device
    f64 = torch.float64
    out = {"o": torch.zeros(b, W + 1, hq, d, dtype=f64, device=dev),
           "lse": torch.zeros(b, W + 1, hq, dtype=f64, device=dev),
           "selected": torch.full((b, hk, k_max), -1, dtype=torch.int32, device=dev),
           "mask": torch.full((b, hk, k_max), -1, dtype=torch.int32, device=dev),
           "num_selected": torch.zeros(b, hk, dtype=torch.int32, device=dev)}
    A, oc, zc = A.clone(), oc.to(f64), zc.to(f64)
    taus = torch.arange(W + 1, device=dev) + (t - W)
    for s in range(b):
        n = keys[s].shape[0]
        lo, hi = _digests(keys[s], P)
        sc = _scores(q[s, W].view(hk, G, d), lo, hi)
        k = _keep(c, n)
        pages = sc.sort(dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
        A[s, :, (n - n_new) // P:(n - 1) // P + 1] = t - 1
        M = A[s].gather(1, pages)
        A[s].scatter_(1, pages, t)
        out["selected"][s, :, :k] = pages.to(torch.int32)
        out["mask"][s, :, :k] = M
        out["num_selected"][s] = k
        for h in range(hk):
            pos = (pages[h][:, None] * P + torch.arange(P, device=dev)).view(-1)
            ok = pos < n
            pos = pos.clamp(max=n - 1)
            K, V = keys[s][pos, h].to(f64), vals[s][pos, h].to(f64)
            Q = q[s, :, h * G:(h + 1) * G].to(f64)                     # [W+1][G][d]
            x = (Q.reshape(-1, d) @ K.t()).view(W + 1, G, -1) / math.sqrt(d)
            use = (M[h][None] < taus[:, None]) | (taus == t)[:, None]  # [W+1][pages]
            use = use.repeat_interleave(P, dim=1) & ok
            x = x.masked_fill(~use[:, None], -math.inf)
            z = torch.logsumexp(x, dim=2)                              # [W+1][G]
            p = torch.exp(x - torch.where(torch.isfinite(z), z, torch.zeros_like(z))[..., None])
            o = (p.view(-1, p.shape[2]) @ V).view(W + 1, G, d)
            heads = slice(h * G, (h + 1) * G)
            for r in range(W):
                co, cz = oc[s, (t - W + r) % W, heads], zc[s, (t - W + r) % W, heads]
                zz = torch.logaddexp(cz, z[r])
                o[r] = torch.exp(cz - zz)[:, None] * co + torch.exp(z[r] - zz)[:, None] * o[r]
                z[r] = zz
            out["o"][s, :, heads] = o
            out["lse"][s, :, heads] = z
    for r in range(W + 1 if W else 0):    # row W last: it takes the slot that row 0 leaves
        oc[:, (t - W + r) % W] = out["o"][:, r]
        zc[:, (t - W + r) % W] = out["lse"][:, r]
    out.update(o_cache=oc, lse_cache=zc, last_loaded=A,
               lens=torch.tensor([x.shape[0] for x in keys], dtype=torch.int32, device=dev))
    return out


def _k_max(c):
    bt = max(c["budget"], _max_pages(c) * c["page"] * c["permille"] // 1000)
    return min(bt // c["page"], _max_pages(c))


def exact(case, seed):
    c = case
    if c["kind"] == "decoder":
        return _exact_stack(c, seed)
    g = _gen(seed)
    if c["kind"] == "prefill":
        return _exact_prefill(c, _layer_inputs(c, g))
    res = []
    for _ in range(c["layers"]):
        x = _layer_inputs(c, g)
        keys, vals = [], []
        for s, (k, v) in enumerate(x["prompt"]):
            if c["update"]:
                m = min(c["window"], k.shape[0])
                k = torch.cat([k[:k.shape[0] - m], x["ku"][0][s, c["window"] - m:]])
                v = torch.cat([v[:v.shape[0] - m], x["vu"][0][s, c["window"] - m:]])
            keys.append(torch.cat([k, x["k"][0][:, s]]))
            vals.append(torch.cat([v, x["v"][0][:, s]]))
        res.append(_exact_step(c, T0, x["q"][0], keys, vals, c["tokens"], x["A"], x["oc"],
                               x["zc"], _k_max(c)))
    return res


def _exact_prefill(c, x):
    b, hk, d, P, mp, td = (c["batch"], c["kv_heads"], c["head_dim"], c["page"], _max_pages(c),
                           _TD[c["dtype"]])
    kc = torch.zeros(b * mp, hk, P, d, dtype=td, device="cuda")
    vc = torch.zeros(b * mp, hk, d, P, dtype=td, device="cuda")
    dg = torch.zeros(b, hk, mp, 2, d, dtype=td, device="cuda")
    for s, (k, v) in enumerate(x["prompt"]):
        pos = torch.arange(k.shape[0], device="cuda")
        ph = x["table"][s].long()[pos // P]
        kc[ph, :, pos % P] = k
        vc[ph, :, :, pos % P] = v
        lo, hi = _digests(k, P)
        dg[s, :, :lo.shape[1], 0], dg[s, :, :lo.shape[1], 1] = lo.to(td), hi.to(td)
    lens = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    return {"k": kc, "v": vc, "digest": dg, "lens": lens}


def _exact_stack(c, seed):
    """The stack in 64 bits, rounded to bf16 where a bf16 stack rounds (projections'
    results, the next layer's input)."""
    weights, per, wins = _stack_inputs(c, seed)
    f64, td, W, b = torch.float64, _TD[c["dtype"]], c["window"], c["batch"]
    hk, hq, d = c["kv_heads"], c["kv_heads"] * c["group"], c["head_dim"]
    low = c["dtype"] == "bf16"

    def rnd(x):
        return x.to(td).to(f64) if low else x

    h = wins[0].to(f64)
    lse = []
    for w, x in zip(weights, per):
        inp = rnd(h)
        q = rnd(inp @ w["wq"].to(f64)).view(b, W + 1, hq, d)
        k = rnd(inp @ w["wk"].to(f64)).view(b, W + 1, hk, d)
        v = rnd(inp @ w["wv"].to(f64)).view(b, W + 1, hk, d)
        keys, vals = [], []
        for s, (pk, pv) in enumerate(x["prompt"]):
            keys.append(torch.cat([pk[:pk.shape[0] - W].to(f64), k[s]]))
            vals.append(torch.cat([pv[:pv.shape[0] - W].to(f64), v[s]]))
        r = _exact_step(c, T0, q, keys, vals, 1, x["A"], x["oc"], x["zc"], _k_max(c))
        y = rnd(rnd(r["o"]).view(b, W + 1, hq * d) @ w["wo"].to(f64))
        # the residual stream is kept in fp32
        h = h + y
        lse.append(r["lse"])
    return {"h": h, "lse": lse,
            "lens": [torch.tensor([n + 1 for n in _lens(c)], dtype=torch.int32, device="cuda")
                     for _ in per]}
