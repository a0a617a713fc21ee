"""Performance cases of the DAR attention library: the calls that a user makes,
over the range of sizes that they are made with.

Four kinds of call, each through the package's public functions:
  prefill  dar_attn_prefill / dar_attn_prefill_rope over whole sequences
  train    the forward with its log-sum-exp, then the backward (plain or rotary)
  decode   one decode step over a cache that holds a long history (dense, or
           paged with a length per sequence; plain or rotary)
  serve    a request over the paged cache: ragged prompts arriving in chunks,
           then single-token append + decode steps

exact() restates the definition (Eq. 1-4 of the paper and, for training, its
gradient by autograd) in plain fp64 torch.
"""
from __future__ import annotations

import math

import torch

import paper_2606_18587_amd as dar

ROPE_BASE = 10000.0
PAGE = 64


def _case(kind, name=None, *, B, Hq, Hkv, T, d, dd, w, dtype="bf16", rope=0, untied=False,
          paged=False, lo=0, chunk=0, steps=0):
    """T: sequence length (decode: cached tokens, serve: prompt length); lo:
    shortest sequence of a ragged batch (0: all hold T)."""
    c = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, T=T, d=d, dd=dd, w=w, dtype=dtype, rope=rope,
             untied=untied, paged=paged, lo=lo, chunk=chunk, steps=steps)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a gradient check or a small fp32 fine-tune: one short sequence in fp32
        _case("train", "train_fp32_short", B=1, Hq=8, Hkv=8, T=331, d=64, dd=16, w=64, dtype="f32"),
        # one short prompt, an odd length: latency
        _case("prefill", "prefill_short", B=1, Hq=8, Hkv=8, T=331, d=64, dd=16, w=128),
        # evaluation batch at the Pythia-70M pretraining shape
        _case("prefill", "prefill_pythia70m", B=8, Hq=8, Hkv=8, T=2048, d=64, dd=16, w=256),
        # one long prompt, grouped queries, head dimension 128
        _case("prefill", "prefill_long16k", B=1, Hq=32, Hkv=8, T=16384, d=128, dd=32, w=1024),
        # the Pythia-410M shape with the rotary embedding inside the attention
        _case("prefill", "prefill_rope_410m", B=4, Hq=16, Hkv=16, T=2048, d=64, dd=16, w=512,
              rope=16),
        # a pretraining step's attention, forward and backward
        _case("train", "train_pythia70m", B=8, Hq=8, Hkv=8, T=2048, d=64, dd=16, w=256),
        # a 1B fine-tune's attention: grouped queries, d = 128, W_up of its own, odd length
        _case("train", "train_gqa_d128", B=2, Hq=16, Hkv=4, T=4001, d=128, dd=32, w=512,
              untied=True),
        # a pretraining step with the rotary embedding
        _case("train", "train_rope_410m", B=4, Hq=16, Hkv=16, T=2048, d=64, dd=16, w=128, rope=16),
        # a full serving batch at 32K tokens of history
        _case("decode", "decode_1b", B=32, Hq=32, Hkv=8, T=32768, d=64, dd=16, w=512),
        # rotary decode of a larger head
        _case("decode", "decode_rope_d128", B=8, Hq=32, Hkv=8, T=16384, d=128, dd=32, w=1024,
              rope=64),
        # continuous batching: sequences of 1K to 32K tokens in pages
        _case("decode", "decode_ragged", B=32, Hq=32, Hkv=8, T=32768, d=64, dd=16, w=512,
              paged=True, lo=1024),
        # a few requests: prompts of 300 to 2600 tokens in chunks of 512, then 16 tokens
        _case("serve", "serve_paged", B=4, Hq=32, Hkv=8, T=2600, d=64, dd=16, w=512, paged=True,
              lo=300, chunk=512, steps=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = {"prefill": 6.0e11, "train": 6.0e11, "decode": 6.0e8, "serve": 6.0e10}
    while True:
        kind = rng.choice(["prefill", "prefill", "train", "train", "decode", "decode", "serve"])
        d = rng.choice([64, 64, 128])
        dd = rng.choice([d // 4, d // 4, 16, 32])
        w = _log_int(rng, 48, 1024)
        Hkv = rng.choice([4, 8, 8, 16])
        Hq = Hkv * rng.choice([1, 1, 2, 4])
        untied = rng.random() < 0.3
        if kind == "prefill":
            c = _case(kind, B=_log_int(rng, 1, 8), Hq=Hq, Hkv=Hkv, T=_log_int(rng, 100, 16384), d=d,
                      dd=dd, w=w, rope=rng.choice([0, 0, 16, 64]), untied=untied)
        elif kind == "train":
            if rng.random() < 0.2:
                c = _case(kind, B=1, Hq=8, Hkv=8, T=_log_int(rng, 64, 360), d=64, dd=16,
                          w=_log_int(rng, 16, 128), dtype="f32", untied=untied)
            else:
                c = _case(kind, B=_log_int(rng, 1, 8), Hq=Hq, Hkv=Hkv, T=_log_int(rng, 200, 4096),
                          d=d, dd=dd, w=w, rope=rng.choice([0, 0, 16]), untied=untied)
        elif kind == "decode":
            paged = rng.random() < 0.5
            T = _log_int(rng, 500, 32768)
            c = _case(kind, B=_log_int(rng, 1, 32), Hq=Hq, Hkv=Hkv, T=T, d=d, dd=dd, w=w,
                      rope=rng.choice([0, 0, 64]), paged=paged, lo=max(1, T // 16) if paged else 0,
                      untied=untied)
        else:
            T = _log_int(rng, 100, 2600)
            c = _case(kind, B=_log_int(rng, 1, 4), Hq=Hq, Hkv=Hkv, T=T, d=d, dd=dd, w=w, paged=True,
                      lo=max(1, T // 8), chunk=rng.choice([128, 256, 512]),
                      steps=rng.choice([4, 8, 16]))
            if -(-c["T"] // c["chunk"]) > 20:
                continue
        wk = work(c)
        # the cost of a case: matrix work, or bytes where a step only streams its cache
        if (wk["bytes"] if kind == "decode" else wk["flops"]) <= most[kind]:
            return c


# --- what a case holds --------------------------------------------------------

def _lens(c):
    """Lengths of a batch's sequences: spread evenly over the logarithm from lo
    to T (all T where lo is 0), in an order that mixes long and short."""
    B, T, lo = c["B"], c["T"], c["lo"]
    if not lo:
        return [T] * B
    if B == 1:
        return [T]
    ls = [int(round(lo * (T / lo) ** (b / (B - 1)))) for b in range(B)]
    step = next(s for s in (13, 11, 7, 5, 3, 2, 1) if math.gcd(s, B) == 1)
    return [ls[(b * step + B - 1) % B] for b in range(B)]


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _inputs(c, seed):
    """Queries, keys, values, weights (and the incoming gradient) of a case."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = _dtype(c)
    B, Hq, Hkv, T, d, dd = (c[x] for x in ("B", "Hq", "Hkv", "T", "d", "dd"))

    def normal(*shape, std=1.0):
        x = torch.randn(*shape, generator=g, device="cuda", dtype=dt)
        return x if std == 1.0 else x * std

    n = T + c["steps"]
    x = {"wd": normal(Hkv, d, dd, std=d ** -0.5),
         "wu": normal(Hkv, dd, d, std=dd ** -0.5) if c["untied"] else None,
         "k": normal(B, Hkv, n, d), "v": normal(B, Hkv, n, d)}
    x["q"] = normal(B, Hq, d) if c["kind"] == "decode" else normal(B, Hq, n, d)
    if c["kind"] == "train":
        x["dout"] = normal(B, Hq, T, d)
    return x


def _paged_cache(c, cap):
    """An empty paged cache whose pages are handed out in a shuffled order."""
    blocks = -(-cap // PAGE)
    cache = dar.DarPagedCache(c["B"], c["Hkv"], c["d"], c["dd"], c["w"], PAGE, blocks,
                              blocks * c["B"], _dtype(c))
    cache.block_table.copy_(_pages(c, blocks))
    return cache


def _pages(c, blocks):
    g = torch.Generator().manual_seed(blocks)
    return torch.randperm(blocks * c["B"], generator=g).reshape(c["B"], blocks).to(torch.int32)


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    s = {"case": c, "wd": x["wd"], "wu": x["wu"]}
    B, Hq, T = c["B"], c["Hq"], c["T"]
    if c["kind"] in ("prefill", "train"):
        s.update({n: x[n] for n in ("q", "k", "v")}, dout=x.get("dout"))
        if c["rope"]:
            s["rope"] = dar.Rope(c["rope"], ROPE_BASE, T)
    elif c["kind"] == "decode" and not c["paged"]:
        cache = dar.DarCache(B, c["Hkv"], c["d"], c["dd"], c["w"], T, _dtype(c))
        dar.dar_cache_append(cache, x["k"], x["v"], x["wd"], Hq=Hq)
        s.update(cache=cache, q=x["q"], rope=dar.Rope(c["rope"], ROPE_BASE, T) if c["rope"] else None)
    elif c["kind"] == "decode":
        cache = _paged_cache(c, T)
        n_new = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
        # the history goes in as prompt chunks (their outputs are not needed)
        done = 0
        while done < T:
            n = min(4096, T - done)
            k, v = (x[a][:, :, done:done + n].contiguous() for a in "kv")
            q = torch.zeros(B, Hq, n, c["d"], dtype=_dtype(c), device="cuda")
            dar.dar_attn_prefill_chunk_paged(cache, q, k, v, x["wd"], x["wu"],
                                             n_new=(n_new - done).clamp(0, n).to(torch.int32))
            done += n
        s.update(cache=cache, q=x["q"],
                 rope=dar.Rope(c["rope"], ROPE_BASE, cache.cap) if c["rope"] else None)
    else:
        s["cache"] = _paged_cache(c, T + c["steps"])
        lens = torch.tensor(_lens(c), dtype=torch.int32)
        s["chunks"] = []
        for at in range(0, T, c["chunk"]):
            n = min(c["chunk"], T - at)
            q, k, v = (x[a][:, :, at:at + n].contiguous() for a in "qkv")
            # rows past a sequence's share of the chunk are not written by the call
            s["chunks"].append((q, k, v, (lens - at).clamp(0, n).to(torch.int32).cuda(),
                                torch.zeros_like(q)))
        s["steps"] = [tuple(x[a][:, :, T + t].contiguous() for a in "qkv")
                      for t in range(c["steps"])]
    return s


def run(state):
    s, c = state, state["case"]
    wd, wu, w = s["wd"], s["wu"], c["w"]
    if c["kind"] == "prefill":
        if c["rope"]:
            return {"o": dar.dar_attn_prefill_rope(s["q"], s["k"], s["v"], wd, wu, w, s["rope"])}
        return {"o": dar.dar_attn_prefill(s["q"], s["k"], s["v"], wd, wu, w)}
    if c["kind"] == "train":
        if c["rope"]:
            o, lse = dar.dar_attn_prefill_rope(s["q"], s["k"], s["v"], wd, wu, w, s["rope"],
                                               return_lse=True)
            g = dar.dar_attn_prefill_rope_backward(s["q"], s["k"], s["v"], wd, wu, w, s["rope"], o,
                                                   lse, s["dout"])
        else:
            o, lse = dar.dar_attn_prefill_lse(s["q"], s["k"], s["v"], wd, wu, w)
            g = dar.dar_attn_prefill_backward(s["q"], s["k"], s["v"], wd, wu, w, o, lse, s["dout"])
        out = {"o": o, "lse": lse, "dq": g[0], "dk": g[1], "dv": g[2], "dw_down": g[3]}
        if g[4] is not None:
            out["dw_up"] = g[4]
        return out
    cache = s["cache"]
    if c["kind"] == "decode":
        if c["paged"]:
            if c["rope"]:
                return {"o": dar.dar_attn_decode_paged_rope(cache, s["q"], wd, s["rope"], wu)}
            return {"o": dar.dar_attn_decode_paged(cache, s["q"], wd, wu)}
        if c["rope"]:
            return {"o": dar.dar_attn_decode_rope(cache, s["q"], wd, s["rope"], wu)}
        return {"o": dar.dar_attn_decode(cache, s["q"], wd, wu)}
    cache.lens.zero_()  # the slots take new requests
    for q, k, v, n_new, o in s["chunks"]:
        dar.dar_attn_prefill_chunk_paged(cache, q, k, v, wd, wu, n_new=n_new, o=o)
    tokens = []
    for q, k, v in s["steps"]:
        dar.dar_cache_append_paged(cache, k, v, wd, Hq=c["Hq"])
        tokens.append(dar.dar_attn_decode_paged(cache, q, wd, wu))
    return {"chunks": [x[4] for x in s["chunks"]], "tokens": tokens, "lens": cache.lens,
            "k_win": cache.k_win, "v_win": cache.v_win, "k_pool": cache.k_pool,
            "v_pool": cache.v_pool}


# --- what a case cannot do without -------------------------------------------

def _pairs(T, w):
    """Causal (query, key) pairs of a sequence: inside the window, beyond it."""
    near = min(T, w)
    local = near * (near + 1) // 2 + (T - near) * w
    return local, T * (T + 1) // 2 - local


def work(case):
    c = case
    B, Hq, Hkv, T, d, dd, w = (c[x] for x in ("B", "Hq", "Hkv", "T", "d", "dd", "w"))
    es = 2 if c["dtype"] == "bf16" else 4
    weights = Hkv * d * dd * es * (2 if c["untied"] else 1)
    # a distant pair: scores and values at d_down (absorbed); with rotation the
    # scores stay at d
    key_d = d if c["rope"] else dd
    if c["kind"] in ("prefill", "train"):
        local, far = (B * Hq * x for x in _pairs(T, w))
        qb, kb = B * Hq * T * d * es, B * Hkv * T * d * es
        flops = 4 * d * local + 2 * (key_d + dd) * far
        nbytes = 2 * qb + 2 * kb + weights
        if c["kind"] == "train":
            # scores again, dP, dV, dK, dQ; beyond the window also O_lat for dW_up
            flops += 10 * d * local + (6 * key_d + 6 * dd) * far
            nbytes += B * Hq * T * 4 + 2 * qb + 2 * kb  # lse, dout, dq, dk, dv
            nbytes += Hkv * d * dd * 4 * (2 if c["untied"] else 1)
        return {"bytes": nbytes, "flops": flops}
    flops = nbytes = 0
    if c["kind"] == "decode":
        for n in _lens(c):
            near = min(n, w)
            nbytes += Hkv * 2 * es * (near * d + (n - near) * dd)
            flops += Hq * (4 * d * near + 2 * (key_d + dd) * (n - near))
        nbytes += 2 * B * Hq * d * es + weights
        return {"bytes": nbytes, "flops": flops}
    for n in _lens(c):
        local, far = _pairs(n, w)
        flops += Hq * (4 * d * local + 4 * dd * far)
        nbytes += 2 * n * (Hq + Hkv) * d * es
        for t in range(c["steps"]):
            m = n + t + 1
            near = min(m, w)
            nbytes += Hkv * 2 * es * (near * d + (m - near) * dd) + 2 * (Hq + Hkv) * d * es
            flops += Hq * (4 * d * near + 4 * dd * (m - near))
        left = max(0, n + c["steps"] - w)
        nbytes += Hkv * 2 * es * (min(n, w) * d + left * dd)
    return {"bytes": nbytes + weights, "flops": flops}


def tolerance(case):
    """About four times the error against exact() (bf16: operands, weights of
    the softmax and results rounded to 8 bits; fp32: sums of up to T terms)."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-4}
    return {"rel": 0.02, "max": 0.4}


# --- the same in 64 bits ------------------------------------------------------

def _rotate(x, r, pos):
    """Rotate-half rotary embedding of rows x [..., n, d] at positions pos [n]."""
    if not r:
        return x
    h = r // 2
    ang = pos.double()[:, None] * ROPE_BASE ** (-torch.arange(h, device=x.device).double() * 2 / r)
    cos, sin = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :h], x[..., h:r]
    return torch.cat([a * cos - b * sin, a * sin + b * cos, x[..., r:]], dim=-1)


def _attend(q, k, v, wd, wu, w, r, pos):
    """Eq. 3-4 for the queries q [n, d] at positions pos [n] of one head over
    its keys and values [T, d]; (o, log-sum-exp)."""
    T, d = k.shape
    at = torch.arange(T, device=k.device)
    qr = _rotate(q, r, pos)
    kw = _rotate(k, r, at)
    kl = _rotate((k @ wd) @ wu, r, at)
    vl = (v @ wd) @ wu
    age = pos[:, None] - at[None, :]
    near = (age < w)
    sc = torch.where(near, qr @ kw.t().contiguous(), qr @ kl.t().contiguous()) / math.sqrt(d)
    sc = sc.masked_fill(age < 0, float("-inf"))
    lse = torch.logsumexp(sc, dim=1)
    p = torch.exp(sc - lse[:, None])
    return (p * near) @ v + (p * ~near) @ vl, lse


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    B, Hq, Hkv, T, d, w, r = (c[a] for a in ("B", "Hq", "Hkv", "T", "d", "w", "rope"))
    G = Hq // Hkv
    wd = x["wd"].double()
    tied = x["wu"] is None
    wu = wd.transpose(1, 2).contiguous() if tied else x["wu"].double()
    dev = wd.device
    if c["kind"] == "train":
        out = {n: torch.zeros(x[s].shape, dtype=torch.float64, device=dev)
               for n, s in (("o", "q"), ("dq", "q"), ("dk", "k"), ("dv", "v"), ("dw_down", "wd"))}
        out["lse"] = torch.zeros(B, Hq, T, dtype=torch.float64, device=dev)
        if not tied:
            out["dw_up"] = torch.zeros_like(wu)
        pos = torch.arange(T, device=dev)
        for b in range(B):
            for h in range(Hq):
                g = h // G
                leaf = [t.double().requires_grad_() for t in (x["q"][b, h], x["k"][b, g],
                                                              x["v"][b, g], x["wd"][g])]
                if tied:
                    up = leaf[3].t()
                else:
                    up = x["wu"][g].double().requires_grad_()
                    leaf.append(up)
                o, lse = _attend(leaf[0], leaf[1], leaf[2], leaf[3], up, w, r, pos)
                gr = torch.autograd.grad(o, leaf, x["dout"][b, h].double())
                out["o"][b, h], out["lse"][b, h] = o.detach(), lse.detach()
                out["dq"][b, h] = gr[0]
                for n, t in (("dk", gr[1]), ("dv", gr[2])):
                    out[n][b, g] += t
                out["dw_down"][g] += gr[3]
                if not tied:
                    out["dw_up"][g] += gr[4]
        return out
    if c["kind"] == "prefill":
        o = torch.zeros(B, Hq, T, d, dtype=torch.float64, device=dev)
        for b in range(B):
            for h in range(Hq):
                g = h // G
                for i in range(0, T, 4096):
                    n = min(4096, T - i)
                    pos = torch.arange(i, i + n, device=dev)
                    o[b, h, i:i + n], _ = _attend(x["q"][b, h, i:i + n].double(),
                                                  x["k"][b, g, :i + n].double(),
                                                  x["v"][b, g, :i + n].double(), wd[g], wu[g], w, r,
                                                  pos)
        return {"o": o}
    lens = _lens(c)
    if c["kind"] == "decode":
        o = torch.zeros(B, Hq, d, dtype=torch.float64, device=dev)
        for b in range(B):
            n = lens[b]
            pos = torch.full((G,), n - 1, device=dev)
            for g in range(Hkv):
                o[b, g * G:(g + 1) * G], _ = _attend(x["q"][b, g * G:(g + 1) * G].double(),
                                                     x["k"][b, g, :n].double(),
                                                     x["v"][b, g, :n].double(), wd[g], wu[g], w, r,
                                                     pos)
        return {"o": o}
    # serve: a sequence's tokens are its prompt, then the decoded ones
    steps, chunk = c["steps"], c["chunk"]
    blocks = -(-(T + steps) // PAGE)
    pages = _pages(c, blocks)
    starts = range(0, T, chunk)
    chunks = [torch.zeros(B, Hq, min(chunk, T - a), d, dtype=torch.float64, device=dev)
              for a in starts]
    tokens = [torch.zeros(B, Hq, d, dtype=torch.float64, device=dev) for _ in range(steps)]
    win = {n: torch.zeros(B, Hkv, max(w, 1), d, dtype=torch.float64, device=dev) for n in "kv"}
    pool = {n: torch.zeros(blocks * B, Hkv, PAGE, c["dd"], dtype=torch.float64, device=dev)
            for n in "kv"}
    for b in range(B):
        n = lens[b]
        total = n + steps
        idx = torch.cat([torch.arange(n), T + torch.arange(steps)]).to(dev)
        rows = {a: x[a][b][:, idx].double() for a in "qkv"}
        pos = torch.arange(total, device=dev)
        for h in range(Hq):
            g = h // G
            o, _ = _attend(rows["q"][h], rows["k"][g], rows["v"][g], wd[g], wu[g], w, 0, pos)
            for j, a in enumerate(starts):
                m = max(0, min(chunk, n - a, T - a))
                chunks[j][b, h, :m] = o[a:a + m]
            for t in range(steps):
                tokens[t][b, h] = o[n + t]
        left = max(0, total - w)
        for a in "kv":
            if w:
                keep = pos[left:]
                win[a][b][:, keep % w] = rows[a][:, left:]
            lat = torch.stack([rows[a][g, :left] @ wd[g] for g in range(Hkv)])
            for j in range(-(-left // PAGE)):
                part = lat[:, j * PAGE:(j + 1) * PAGE]
                pool[a][int(pages[b, j]), :, :part.shape[1]] = part
    return {"chunks": chunks, "tokens": tokens, "lens": None, "k_win": win["k"], "v_win": win["v"],
            "k_pool": pool["k"], "v_pool": pool["v"]}
