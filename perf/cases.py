"""Measured cases of the refusal-gated decoding library.

Each case is a plain dict; `prepare` builds what a serving program holds before
the call (weights behind a model handle, KV buffers, logits), `run` makes one
pass through the public entry points of `paper_2607_20791_amd`, and `exact`
computes the same outputs in 64-bit torch from the inputs alone.

Kinds:
  sample     min-p draws on given logits (a server that owns its model and uses the sampler alone)
  pless      p-less draws on given logits
  attention  decode attention of one layer over shared prompts plus paged tails
  lm_head    the LM head on given hidden states
  prefill    prompts through every layer into the shared KV, in chunks of max_rows tokens
  gate       last prompt token over a resident prefix, greedy probe against a refusal table, gate
  decode     N sampled continuations of every prompt over a resident prefix
  generate   prefill and sampled continuations of a small fp32 decoder

Model weights are random.  The embedding has standard deviation 2 and the LM
head's row next(t) is the embedding of t, scaled, for a random cyclic order
`next`: as in a trained model the next token then stands clear of the rest (by
more than the widest truncation window used here), so token sequences do not
hang on the last bit of a logit, and refusal prefixes can be written down.
"""
import math

import numpy as np
import torch

import paper_2607_20791_amd as rgd

PAGE = 16
D = 128  # head dimension of the bf16 models


def listed():
    return [
        # one request's next token: launches and latency
        {"name": "sample-1x128256", "kind": "sample", "rows": 1, "vocab": 128256, "T": 1.0, "min_p": 0.1},
        # the sampler sweep's rows: a full batch at the largest vocabulary
        {"name": "sample-256x152064", "kind": "sample", "rows": 256, "vocab": 152064, "T": 1.5, "min_p": 0.1},
        # the truncation the paper samples with, one prompt's 64 branches
        {"name": "pless-64x128256", "kind": "pless", "rows": 64, "vocab": 128256, "T": 1.5},
        # 64 branches over one long prompt, half way through their tokens
        {"name": "attention-1x64-p8193", "kind": "attention", "prompts": 1, "branches": 64, "heads": 32,
         "kv_heads": 8, "prefix": 8193, "tail": 64},
        # a batch of prompts with 8 branches each, late in their tokens
        {"name": "attention-32x8-p1024", "kind": "attention", "prompts": 32, "branches": 8, "heads": 32,
         "kv_heads": 8, "prefix": 1024, "tail": 200},
        # the head of one 64-branch step
        {"name": "lm_head-64", "kind": "lm_head", "rows": 64, "d": 4096, "vocab": 128256},
        # one prompt refused to the end of the probe: 15 one-row steps
        {"name": "gate-1-p8192", "kind": "gate", "layers": 1, "d": 4096, "ffn": 14336, "heads": 32, "kv_heads": 8,
         "vocab": 128256, "prompts": 1, "prefix": 8192, "k": 16, "hits": 1},
        # 64 branches of one long prompt
        {"name": "decode-1x64-p8192", "kind": "decode", "layers": 1, "d": 4096, "ffn": 14336, "heads": 32,
         "kv_heads": 8, "vocab": 128256, "prompts": 1, "branches": 64, "prefix": 8193, "steps": 8, "T": 2.0,
         "min_p": 0.05},
        # the ungated batch: 32 prompts, 8 branches each
        {"name": "decode-32x8-p1024", "kind": "decode", "layers": 2, "d": 4096, "ffn": 14336, "heads": 32,
         "kv_heads": 8, "vocab": 128256, "prompts": 32, "branches": 8, "prefix": 1024, "steps": 4, "T": 2.0,
         "min_p": 0.1},
        # prompts into the KV of a server that steps 256 rows at a time, ragged last segment
        {"name": "prefill-8x1000-r256", "kind": "prefill", "layers": 2, "d": 4096, "ffn": 14336, "heads": 32,
         "kv_heads": 8, "vocab": 128256, "prompts": 8, "tokens": 1000, "max_rows": 256},
        # one long prompt in large chunks
        {"name": "prefill-1x4096-r2048", "kind": "prefill", "layers": 1, "d": 4096, "ffn": 14336, "heads": 32,
         "kv_heads": 8, "vocab": 128256, "prompts": 1, "tokens": 4096, "max_rows": 2048},
        # the small fp32 decoder: 16 prompts of 64 tokens, 32 tokens each
        {"name": "generate-f32-16x64", "kind": "generate", "layers": 2, "d": 256, "ffn": 1024, "heads": 4,
         "kv_heads": 2, "head_dim": 64, "vocab": 8192, "prompts": 16, "tokens": 64, "branches": 1, "steps": 32,
         "T": 2.0, "min_p": 0.1},
    ]


def _log(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["sample", "pless", "attention", "lm_head", "prefill", "gate", "decode", "generate"])
    d = rng.choice([1024, 2048, 3072, 4096])
    shape = {"layers": rng.choice([1, 2]), "d": d, "ffn": rng.choice([11, 14]) * d // 4 // 128 * 128,
             "heads": d // D, "kv_heads": rng.choice([d // D // 4, d // D // 2]),
             "vocab": 128 * rng.randint(250, 1002)}
    if kind in ("sample", "pless"):
        c = {"kind": kind, "rows": _log(rng, 1, 256), "vocab": 4 * _log(rng, 8000, 38016),
             "T": rng.choice([0.7, 1.0, 1.5, 2.0, 3.0])}
        if kind == "sample":
            c["min_p"] = rng.choice([0.05, 0.1, 0.2])
        return c
    if kind == "attention":
        prompts = _log(rng, 1, 32)
        kv_heads = rng.choice([4, 8])
        return {"kind": kind, "prompts": prompts, "branches": _log(rng, 1, 256 // prompts),
                "heads": kv_heads * rng.choice([1, 2, 4, 8]), "kv_heads": kv_heads,
                "prefix": _log(rng, 60, 8193 if prompts < 8 else 2048), "tail": rng.randint(0, 256)}
    if kind == "lm_head":
        return {"kind": kind, "rows": _log(rng, 1, 256), "d": d, "vocab": shape["vocab"]}
    if kind == "prefill":
        prompts = _log(rng, 1, 8)
        tokens = _log(rng, 30, 4096 // prompts)
        return {"kind": kind, **shape, "prompts": prompts, "tokens": tokens,
                "max_rows": rng.choice([64, 256, 1024, 2048])}
    if kind == "gate":
        prompts = _log(rng, 1, 32)
        return {"kind": kind, **shape, "prompts": prompts, "prefix": _log(rng, 60, 8192 if prompts < 8 else 2048),
                "k": _log(rng, 2, 16), "hits": rng.randint(0, prompts)}
    if kind == "decode":
        prompts = _log(rng, 1, 32)
        return {"kind": kind, **shape, "prompts": prompts, "branches": _log(rng, 1, 256 // prompts),
                "prefix": _log(rng, 60, 8193 if prompts < 8 else 2048), "steps": rng.randint(2, 4),
                "T": rng.choice([1.0, 1.5, 2.0]), "min_p": rng.choice([0.05, 0.1, 0.2])}
    d = rng.choice([128, 256, 512])
    return {"kind": kind, "layers": rng.choice([1, 2]), "d": d, "ffn": 4 * d, "heads": d // 64,
            "kv_heads": max(1, d // 128), "head_dim": 64, "vocab": 4 * _log(rng, 500, 2048),
            "prompts": _log(rng, 1, 16), "tokens": _log(rng, 5, 80), "branches": rng.randint(1, 2),
            "steps": rng.randint(2, 32), "T": rng.choice([1.0, 2.0]), "min_p": 0.1}


# ------------------------------------------------------------------- inputs --
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _normal(g, shape, std, dtype):
    """N(0, std^2) of the given type (drawn in parts: large weights need no fp32 copy)."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        part = flat[i:i + (1 << 27)]
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda").mul_(std))
    return out


def _logits(g, rows, vocab):
    """Rows of fp32 logits: N(0, 1) plus a Zipf(1.1) rank bias of 12 over a random order of the ids."""
    r = torch.arange(1, vocab + 1, device="cuda", dtype=torch.float64)
    vs = float(vocab) ** -1.1
    bias = (12.0 * (r ** -1.1 - vs) / (1.0 - vs)).float()
    z = torch.randn(rows, vocab, generator=g, device="cuda")
    for i in range(rows):
        z[i] += bias[torch.randperm(vocab, generator=g, device="cuda")]
    return z


def _dims(c):
    hd = c.get("head_dim", D)
    dt = torch.float32 if "head_dim" in c else torch.bfloat16
    return c["d"], c["ffn"], c["heads"], c["kv_heads"], hd, c["vocab"], dt


def _weights(c, g):
    """Embedding, LM head, layers, and next: the token that follows each token."""
    d, f, hq, hk, hd, V, dt = _dims(c)
    embed = _normal(g, (V, d), 2.0, dt)
    order = torch.randperm(V, generator=g, device="cuda")
    nxt = torch.empty_like(order)
    nxt[order] = order.roll(-1)
    prev = torch.empty_like(order)
    prev[nxt] = torch.arange(V, device="cuda")
    head = torch.empty_like(embed)
    for i in range(0, V, 16384):
        head[i:i + 16384] = embed[prev[i:i + 16384]] * (16.0 / d)
    layers = []
    for _ in range(c["layers"]):
        L = {"attn_norm": torch.ones(d, device="cuda"), "ffn_norm": torch.ones(d, device="cuda")}
        for n, shp in (("wq", (hq * hd, d)), ("wk", (hk * hd, d)), ("wv", (hk * hd, d)), ("wo", (d, hq * hd)),
                       ("w_gate", (f, d)), ("w_up", (f, d)), ("w_down", (d, f))):
            L[n] = _normal(g, shp, 0.02, dt)
        layers.append(L)
    return {"embed": embed, "final_norm": torch.ones(d, device="cuda"), "lm_head": head}, layers, nxt


def _model(c, top, layers, max_rows, max_pos):
    d, f, hq, hk, hd, V, dt = _dims(c)
    cfg = rgd.ModelConfig(c["layers"], d, hq, hk, hd, f, V,
                          rgd.DTYPE_F32 if dt == torch.float32 else rgd.DTYPE_BF16, 1e-5, 500000.0, max_pos)
    return rgd.Model(cfg, top, layers, max_rows)


def _vp(p):
    return (p + 63) // 64 * 64


def _kv_buffers(layers, prompts, prefix, pages, hk, hd, dt):
    z = lambda *s: torch.zeros(s, dtype=dt, device="cuda")  # noqa: E731
    return (z(layers, prompts, hk, prefix, hd), z(layers, prompts, hk, _vp(prefix) // 64, hd, 64),
            z(layers, max(pages, 1), hk, PAGE, hd), z(layers, max(pages, 1), hk, hd, PAGE))


def _v_blocks(v):
    """[..., P, D] -> the V cache layout [..., VP/64, D, 64], zeros past P."""
    P, hd = v.shape[-2:]
    pad = torch.zeros(v.shape[:-2] + (_vp(P), hd), dtype=v.dtype, device=v.device)
    pad[..., :P, :] = v
    return pad.view(v.shape[:-2] + (_vp(P) // 64, 64, hd)).transpose(-1, -2).contiguous()


def _inputs(c, seed):
    """Everything drawn from the seed, on the GPU, without the library."""
    g = _gen(seed)
    k = c["kind"]
    if k in ("sample", "pless"):
        return {"z": _logits(g, c["rows"], c["vocab"]), "seeds": int(seed) * 1000003 + torch.arange(c["rows"], device="cuda")}
    if k == "lm_head":
        return {"h": _normal(g, (c["rows"], c["d"]), 1.0, torch.bfloat16),
                "w": _normal(g, (c["vocab"], c["d"]), 0.02, torch.bfloat16)}
    if k == "attention":
        R, hk, P, n = c["prompts"] * c["branches"], c["kv_heads"], c["prefix"], -(-c["tail"] // PAGE)
        bf = torch.bfloat16
        return {"q": _normal(g, (R, c["heads"], D), 1.0, bf), "k": _normal(g, (c["prompts"], hk, P, D), 1.0, bf),
                "v": _normal(g, (c["prompts"], hk, P, D), 1.0, bf),
                "tk": _normal(g, (max(R * n, 1), hk, PAGE, D), 1.0, bf),
                "tv": _normal(g, (max(R * n, 1), hk, D, PAGE), 1.0, bf),
                "pages": torch.randperm(max(R * n, 1), generator=g, device="cuda").to(torch.int32).view(-1, max(n, 1))}
    top, layers, nxt = _weights(c, g)
    x = {"top": top, "layers": layers, "next": nxt}
    n = {"prefill": c.get("tokens"), "generate": c.get("tokens")}.get(k, 1)
    x["tokens"] = torch.randint(0, c["vocab"], (c["prompts"], n), generator=g, device="cuda", dtype=torch.int32)
    if k in ("gate", "decode"):  # a resident prefix: rotated keys and values of N(0, 1)
        _, _, _, hk, hd, _, dt = _dims(c)
        P = c["prefix"]
        x["k"] = _normal(g, (c["layers"], c["prompts"], hk, P, hd), 1.0, dt)
        x["v"] = _normal(g, (c["layers"], c["prompts"], hk, P, hd), 1.0, dt)
    if k == "decode":  # the prompts' last logits, as their prefill left them
        x["last"] = torch.randn(c["prompts"], c["vocab"], generator=g, device="cuda")
        x["last"].scatter_(1, x["tokens"].long(), 40.0)
    return x


def _rows(c):
    return c["prompts"] * c["branches"]


def _seeds(c, seed):
    return int(seed) * 1000003 + torch.arange(_rows(c), device="cuda")


# ------------------------------------------------------------------ prepare --
def prepare(case, seed):
    c, k = case, case["kind"]
    x = _inputs(c, seed)
    if k in ("sample", "pless"):
        R, V = x["z"].shape
        return {**x, "c": c, "out": torch.empty(R, 1, dtype=torch.int32, device="cuda"),
                "ws": torch.empty(rgd.sampler_workspace_bytes(R, V), dtype=torch.uint8, device="cuda")}
    if k == "lm_head":
        m = dict(c, layers=1, ffn=128, heads=1, kv_heads=1)
        one = _weights(dict(m, vocab=128), _gen(seed))
        top = {"embed": x["w"], "final_norm": one[0]["final_norm"], "lm_head": x["w"]}
        return {"c": c, "h": x["h"], "model": _model(m, top, one[1], c["rows"], 64),
                "logits": torch.empty(c["rows"], c["vocab"], device="cuda")}
    if k == "attention":
        R = _rows(c)
        m = dict(c, layers=1, d=128, ffn=128, vocab=128)
        top, layers, _ = _weights(m, _gen(seed))
        return {"c": c, "q": x["q"], "k": x["k"], "v": _v_blocks(x["v"]), "tk": x["tk"], "tv": x["tv"],
                "pages": x["pages"], "model": _model(m, top, layers, R, c["prefix"] + 256),
                "prompt": np.repeat(np.arange(c["prompts"], dtype=np.int32), c["branches"]),
                "plen": np.full(R, c["prefix"], np.int32),
                "out": torch.empty(R, c["heads"] * D, dtype=torch.bfloat16, device="cuda")}
    B, V = c["prompts"], c["vocab"]
    _, _, _, hk, hd, _, dt = _dims(c)
    s = {"c": c, "tokens": x["tokens"], "last": torch.empty(B, V, device="cuda")}
    if k == "prefill":
        s["model"] = _model(c, x["top"], x["layers"], c["max_rows"], c["tokens"])
        buf = _kv_buffers(c["layers"], B, c["tokens"], 0, hk, hd, dt)
        s["kv"] = rgd.KV(s["model"], B, c["tokens"], 0, PAGE, *buf)
        return s
    if k == "generate":
        R, n, S = _rows(c), c["tokens"], c["steps"]
        pages = R * (-(-(S - 1) // PAGE))
        s["model"] = _model(c, x["top"], x["layers"], max(R, B * n), n + S)
        s["kv"] = rgd.KV(s["model"], B, n, pages, PAGE, *_kv_buffers(c["layers"], B, n, pages, hk, hd, dt))
    else:
        P = c["prefix"] + (k == "gate")
        R, S = (_rows(c), c["steps"]) if k == "decode" else (B, c["k"])
        pages = R * (-(-(S - 1) // PAGE))
        s["model"] = _model(c, x["top"], x["layers"], R, P + S)
        buf = _kv_buffers(c["layers"], B, P, pages, hk, hd, dt)
        buf[0][:, :, :, :c["prefix"]] = x["k"]
        vb = _v_blocks(x["v"])
        buf[1][:, :, :, :vb.shape[3]] = vb
        s["kv"] = rgd.KV(s["model"], B, P, pages, PAGE, *buf)
    if k == "gate":
        s["table"] = rgd.Table(*_table(c, x), min_match=2)
        s["ptok"] = torch.empty(B, c["k"], dtype=torch.int32, device="cuda")
        s["plen"] = torch.empty(B, dtype=torch.int32, device="cuda")
        s["event"] = torch.empty(B, dtype=torch.int32, device="cuda")
        return s
    if k == "decode":
        s["last"] = x["last"]
        for b in range(B):
            s["kv"].set_prefix_len(b, c["prefix"])
    R = _rows(c)
    s["seeds"] = _seeds(c, seed)
    s["tap"] = torch.empty(c["steps"], R, V, device="cuda")
    s["out"] = torch.empty(B, c["branches"], c["steps"], dtype=torch.int32, device="cuda")
    return s


def _chain(nxt, tokens, n):
    """The n tokens that follow each prompt's last one."""
    t, out = tokens[:, -1].long(), []
    for _ in range(n):
        t = nxt[t]
        out.append(t)
    return torch.stack(out, 1)


def _table(c, x):
    """64 refusal prefixes of 3-6 tokens: the first 4 greedy tokens of the first `hits` prompts, the rest unlike any probe."""
    chain = _chain(x["next"], x["tokens"], 6).cpu().numpy()
    entries = [chain[b, :4] for b in range(c["hits"])]
    entries += [(chain[i % c["prompts"], :3 + i % 4] + 1 + i) % c["vocab"] for i in range(64 - c["hits"])]
    off = np.zeros(len(entries) + 1, np.int32)
    off[1:] = np.cumsum([len(e) for e in entries])
    return off, np.concatenate(entries).astype(np.int32)


# ---------------------------------------------------------------------- run --
def run(state):
    s, c = state, state["c"]
    k = c["kind"]
    if k == "sample":
        rgd.kernel_sample(s["z"], c["T"], c["min_p"], s["seeds"], 3, 0, 1, s["ws"], s["out"])
        return s["out"]
    if k == "pless":
        rgd.kernel_sample_pless(s["z"], c["T"], s["seeds"], 3, 0, 1, s["ws"], s["out"])
        return s["out"]
    if k == "lm_head":
        rgd.kernel_lm_head(s["model"], s["h"], s["logits"])
        return s["logits"]
    if k == "attention":
        rgd.kernel_attention(s["model"], s["q"], s["prompt"], s["plen"], s["k"], s["v"], c["prompts"], c["prefix"],
                             s["tk"], s["tv"], PAGE, s["pages"], s["pages"].shape[1], c["tail"], s["out"])
        return s["out"]
    kv, B = s["kv"], c["prompts"]
    if k in ("prefill", "generate", "gate"):
        start = c.get("prefix", 0)
        for b in range(B):
            kv.set_prefix_len(b, start)
        rgd.prefill_kv(s["model"], kv, s["tokens"], start, s["last"])
    if k == "prefill":
        return {"last": s["last"], "k": kv.prefix_k, "v": kv.prefix_v}
    if k == "gate":
        rgd.probe(s["model"], kv, s["last"], s["table"], B, c["k"], 3, -1, s["ptok"], s["plen"], s["event"])
        hit, miss = rgd.gate(kv, s["event"], B)
        return {"last": s["last"], "tokens": s["ptok"], "len": s["plen"], "event": s["event"], "hit": hit, "miss": miss}
    rgd.sample_continuations(s["model"], kv, s["last"], list(range(B)), c["branches"], c["steps"], c["T"], c["min_p"],
                             s["seeds"], s["out"], logits_tap=s["tap"])
    return {"last": s["last"], "logits": s["tap"], "tokens": s["out"]}


# --------------------------------------------------------------------- work --
def _linear(c):
    """Weights of one layer."""
    d, f, hq, hk, hd, _, _ = _dims(c)
    return d * (hq + 2 * hk) * hd + hq * hd * d + 3 * d * f


def _attn(c, rows, positions):
    """Operations of `rows` rows over a mean of `positions` positions, one layer."""
    _, _, hq, _, hd, _, _ = _dims(c)
    return 4.0 * rows * hq * hd * positions


def work(case):
    c, k = case, case["kind"]
    if k in ("sample", "pless"):
        n = c["rows"] * c["vocab"]
        return {"bytes": 4 * n + 12 * c["rows"], "flops": 4 * n}
    if k == "lm_head":
        return {"bytes": 2 * c["vocab"] * c["d"] + c["rows"] * (2 * c["d"] + 4 * c["vocab"]),
                "flops": 2.0 * c["rows"] * c["d"] * c["vocab"]}
    if k == "attention":
        R, hk = _rows(c), c["kv_heads"]
        return {"bytes": 4 * D * (c["prompts"] * hk * c["prefix"] + R * hk * c["tail"] + R * c["heads"]),
                "flops": 4.0 * R * c["heads"] * D * (c["prefix"] + c["tail"])}
    d, f, hq, hk, hd, V, dt = _dims(c)
    e, L, B = (4 if dt == torch.float32 else 2), c["layers"], c["prompts"]
    lin, head, pos = L * _linear(c), V * d, 2 * L * hk * hd  # weights; K and V values of one position

    def prefill(n, start):
        tok = B * n
        return (e * (lin + head + tok * (d + pos) + B * start * pos) + 4 * B * V,
                2.0 * tok * lin + 2.0 * B * head + L * _attn(c, tok, start + (n + 1) / 2))

    def steps(rows, n, prefix, weights):
        """n decode steps of `rows` rows over B resident prefixes and their own tails, logits written and read."""
        tail = (n + 1) / 2
        return (n * (e * (weights + B * prefix * pos + rows * (d + tail * pos)) + 8 * rows * V),
                n * (2.0 * rows * weights + L * _attn(c, rows, prefix + tail)))

    if k == "prefill":
        b, o = prefill(c["tokens"], 0)
    elif k == "gate":
        b, o = prefill(1, c["prefix"])
        if c["hits"] and c["k"] > 1:  # the prompts that hit decode k - 1 tokens
            b2, o2 = steps(c["hits"], c["k"] - 1, c["prefix"] + 1, lin + head)
            b, o = b + b2 * 1.0, o + o2
    elif k == "decode":
        b, o = steps(_rows(c), c["steps"] - 1, c["prefix"], lin + head)
        b += 8 * _rows(c) * V
    else:
        b, o = prefill(c["tokens"], 0)
        b2, o2 = steps(_rows(c), c["steps"] - 1, c["tokens"], lin + head)
        b, o = b + b2, o + o2
    return {"bytes": float(b), "flops": float(o)}


def tolerance(case):
    k = case["kind"]
    if k in ("sample", "pless"):  # draws that fall on the edge of a token's interval
        return {"rel": 0.0, "differ": 0.01}
    # four times the distance from 64 bits that was measured
    if k in ("lm_head", "generate"):  # fp32 sums: 4e-7
        return {"rel": 2e-6, "differ": 0.0}
    if k == "attention":  # bf16 probabilities, partial outputs and output: 2.8e-3
        return {"rel": 1.1e-2}
    return {"rel": 1.5e-2, "differ": 0.0}  # bf16 activations between kernels: 3.8e-3


# -------------------------------------------------------------------- exact --
def _mm(x, w):
    """x W^T in 64 bits, W in parts."""
    out = torch.empty(x.shape[0], w.shape[0], dtype=torch.float64, device="cuda")
    for i in range(0, w.shape[0], 16384):
        out[:, i:i + 16384] = x @ w[i:i + 16384].double().t()
    return out


def _norm(x):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5)


def _rope(x, pos):
    """Rotate-half rotary embedding of [T][H][D] at positions [T]."""
    hd = x.shape[-1]
    f = 500000.0 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device="cuda") / hd)
    a = (pos.double()[:, None] * f)[:, None, :]
    lo, hi = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _softmax_v(q, k, v, mask):
    """[H][T][D] queries over [H][P][D] keys and values."""
    s = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if mask is not None:
        s.masked_fill_(mask, -math.inf)
    return torch.bmm(torch.softmax(s, -1), v)


class _Exact:
    """The decoder in 64 bits; one K/V history [Hkv][P][D] per (layer, sequence)."""

    def __init__(self, c, x):
        self.c, self.x = c, x
        self.dims = _dims(c)

    def forward(self, tokens, hist, start):
        """tokens [S][T] of S sequences at positions start.., appended to hist[layer][sequence]; last hidden rows."""
        d, _, hq, hk, hd, _, _ = self.dims
        S, T = tokens.shape
        h = self.x["top"]["embed"][tokens.reshape(-1).long()].double()
        pos = start + torch.arange(T, device="cuda")
        G = hq // hk
        for l, L in enumerate(self.x["layers"]):
            n = _norm(h)
            q, k, v = (_mm(n, L[w]).view(S, T, -1, hd) for w in ("wq", "wk", "wv"))
            att = torch.empty(S, T, hq * hd, dtype=torch.float64, device="cuda")
            for s in range(S):
                kk, vv = _rope(k[s], pos).transpose(0, 1), v[s].transpose(0, 1)
                old = hist[l][s]
                if old is not None:
                    kk, vv = torch.cat([old[0].double(), kk], 1), torch.cat([old[1].double(), vv], 1)
                hist[l][s] = (kk, vv)
                P = kk.shape[1]
                mask = torch.arange(P, device="cuda")[None, :] > pos[:, None] if T > 1 else None
                qq = _rope(q[s], pos).transpose(0, 1).reshape(hk, G, T, hd)
                for g in range(hk):
                    kg, vg = kk[g].expand(G, P, hd).contiguous(), vv[g].expand(G, P, hd).contiguous()
                    o = _softmax_v(qq[g].contiguous(), kg, vg, mask)  # [G][T][D]
                    att[s, :, g * G * hd:(g + 1) * G * hd] = o.transpose(0, 1).reshape(T, G * hd)
            h = h + _mm(att.view(S * T, -1), L["wo"])
            n = _norm(h)
            gate = _mm(n, L["w_gate"])
            act = gate * torch.sigmoid(gate) * _mm(n, L["w_up"])
            h = h + _mm(act, L["w_down"])
        return _norm(h).view(S, T, d)[:, -1]

    def logits(self, h):
        return _mm(h, self.x["top"]["lm_head"])


def exact(case, seed):
    c, k = case, case["kind"]
    if k in ("sample", "pless"):
        return None  # the outputs are tokens
    x = _inputs(c, seed)
    if k == "lm_head":
        return _mm(x["h"].double(), x["w"])
    if k == "attention":
        R, hq, hk, G = _rows(c), c["heads"], c["kv_heads"], c["heads"] // c["kv_heads"]
        out = torch.empty(R, hq, D, dtype=torch.float64, device="cuda")
        t = c["tail"]
        for r in range(R):
            kk, vv = x["k"][r // c["branches"]].double(), x["v"][r // c["branches"]].double()
            if t:
                pg = x["pages"][r].long()
                kk = torch.cat([kk, x["tk"][pg].transpose(0, 1).reshape(hk, -1, D)[:, :t].double()], 1)
                vv = torch.cat([vv, x["tv"][pg].permute(1, 0, 3, 2).reshape(hk, -1, D)[:, :t].double()], 1)
            out[r] = _softmax_v(x["q"][r].view(hk, G, D).double(), kk, vv, None).view(hq, D)
        return out.view(R, hq * D)
    m = _Exact(c, x)
    B, L = c["prompts"], c["layers"]
    if k == "gate":
        hist = [[(x["k"][l, b], x["v"][l, b]) for b in range(B)] for l in range(L)]
        last = m.logits(m.forward(x["tokens"], hist, c["prefix"]))
        return {"last": last, "tokens": None, "len": None, "event": None, "hit": None, "miss": None}
    if k in ("prefill", "generate"):
        n = c["tokens"]
        hist = [[None] * B for _ in range(L)]
        last = m.logits(m.forward(x["tokens"], hist, 0))
        kk = torch.stack([torch.stack([hist[l][b][0] for b in range(B)]) for l in range(L)])
        if k == "prefill":
            vv = torch.stack([torch.stack([hist[l][b][1] for b in range(B)]) for l in range(L)])
            return {"last": last, "k": kk, "v": _v_blocks(vv)}
        start = n
    else:
        hist = [[(x["k"][l, b], x["v"][l, b]) for b in range(B)] for l in range(L)]
        last, start = x["last"].double(), c["prefix"]
    # every branch of a prompt draws the same tokens: the next one stands clear of the truncation window
    N = c["branches"]
    z, taps = last, [last]
    for s in range(c["steps"] - 1):
        z = m.logits(m.forward(z.argmax(-1, keepdim=True), hist, start + s))
        taps.append(z)
    return {"last": last, "logits": torch.stack([t.repeat_interleave(N, 0) for t in taps]), "tokens": None}
