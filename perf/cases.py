"""Workloads of this framework, measured through its public entry points.

Four kinds, each a call (or the short chain of calls) that a serving program
makes:

* ``step``       one scheduling round's attention step, ``step_mixed``: the
                 round's K/V rows are appended to the paged pools and its
                 prefill chunks and decode rows attend over them.
* ``attn_proj``  the projections around the step of one decoder layer:
                 RMSNorm, the fused QKV projection, the split with per-head
                 norm and rotary embedding, and the output projection with
                 the residual.
* ``ffn``        the feed-forward block of one decoder layer: RMSNorm,
                 gate/up projection, SwiGLU, down projection with the residual.
* ``model``      a whole iteration of a few decoder layers over one mixed
                 batch, with the logits of each row's last token.

A case is a dict of plain values; row lengths follow from the case (its
``rows_seed``), tensor contents and the placement of pages from the seed.
"""

import math

import numpy as np
import torch

import paper_2606_09061_amd as cp
from paper_2606_09061_amd import model as M

DEV = "cuda:0"
EPS, THETA = 1e-6, 1e6


# ---------------------------------------------------------------- the cases

def _step(hq, hkv, d, block, decodes, median, longest, chunks, rows_seed, long_share=0.0):
    """``chunks``: prefill chunks as "length@prior ..."; ``decodes`` decode rows
    of log-normal context (median, sigma 1, at most ``longest``), of which
    ``long_share`` are uniform up to ``longest`` instead."""
    return {"kind": "step", "hq": hq, "hkv": hkv, "d": d, "block": block, "decodes": decodes,
            "median": median, "longest": longest, "long_share": long_share, "chunks": chunks,
            "rows_seed": rows_seed}


def _named(name, case):
    return {"name": name, **case}


def listed():
    return [
        # the smallest step: a few short rows on few heads; launches and latency
        _named("step-tiny", _step(4, 2, 64, 16, 2, 100, 200, "64@0 48@128", 1)),
        # a lightly loaded server: 8 decode rows, no prefill
        _named("step-decode-8", _step(32, 8, 128, 16, 8, 1024, 8192, "", 2)),
        # an ordinary mixed round under a 512-token budget: decode rows first,
        # two prefill chunks in the rest
        _named("step-budget-512", _step(32, 8, 128, 16, 128, 1024, 8192, "192@1817 192@3391", 3)),
        # a prefill-heavy round under a 2,048-token budget, long prior contexts
        _named("step-prefill-2048", _step(32, 8, 128, 16, 128, 2048, 32768,
                                          "480@0 480@8192 480@16384 480@31744", 4)),
        # a decode-dominated round with long contexts, the largest traffic
        _named("step-decode-256", _step(32, 8, 128, 16, 256, 512, 32768, "256@0", 5, 0.3)),
        # a round of the 64/8-head replay: whole prompts of ragged length
        _named("step-replay-4096", _step(64, 8, 128, 32, 40, 1000, 4096,
                                         "460@0 1161@0 1188@0 1247@0", 6)),
        # a decode batch's projections: weights streamed for a few rows
        _named("proj-decode-24", {"kind": "attn_proj", "tokens": 24, "hidden": 4096, "hq": 32,
                                  "hkv": 8, "d": 128}),
        # a prefill round's projections: large matrix products
        _named("proj-prefill-2048", {"kind": "attn_proj", "tokens": 2048, "hidden": 4096, "hq": 32,
                                     "hkv": 8, "d": 128}),
        # one request decoding: the feed-forward weights streamed for one row
        _named("ffn-decode-1", {"kind": "ffn", "tokens": 1, "hidden": 4096, "inter": 12288}),
        # a busy decode batch: still bound by the weights
        _named("ffn-decode-96", {"kind": "ffn", "tokens": 96, "hidden": 4096, "inter": 12288}),
        # a ragged prefill round: large matrix products, a last row block that
        # is not full
        _named("ffn-prefill-1000", {"kind": "ffn", "tokens": 1000, "hidden": 4096,
                                    "inter": 12288}),
        # a whole iteration of a 4-layer model: 64 decode rows and one chunk
        _named("model-mixed-261", {"kind": "model", "layers": 4, "decodes": 64, "median": 1024,
                                   "longest": 4096, "chunk": 197, "prior": 512, "rows_seed": 7}),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _draw_step(rng):
    hq, hkv, d, block = rng.choice([(4, 2, 64, 16), (32, 8, 128, 16), (32, 8, 128, 16),
                                    (64, 8, 128, 32), (64, 8, 128, 32), (8, 1, 128, 32)])
    chunks, left = [], 4096
    for _ in range(rng.choice([0, 1, 1, 2, 3, 4])):
        c = min(left, _log_int(rng, 2, 2048))
        if c >= 2:
            prior = 0 if rng.random() < 0.5 else _log_int(rng, 1, 16384)
            chunks.append("%d@%d" % (c, prior))
            left -= c
    decodes = _log_int(rng, 1, 256) if (not chunks or rng.random() < 0.8) else 0
    return _step(hq, hkv, d, block, decodes, _log_int(rng, 128, 2048), rng.choice([4096, 8192]),
                 " ".join(chunks), rng.randrange(1 << 30))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "attn_proj", "attn_proj", "ffn", "ffn", "model"])
    if kind == "step":
        while True:
            case = _draw_step(rng)
            w = work(case)  # no dearer than the largest listed steps
            if w["bytes"] <= 4.5e9 and w["flops"] <= 4e11:
                return case
    hidden, hq, hkv, inter = rng.choice([(4096, 32, 8, 12288), (4096, 32, 8, 12288),
                                         (2048, 16, 4, 6144)])
    if kind == "attn_proj":
        return {"kind": kind, "tokens": _log_int(rng, 1, 2040), "hidden": hidden, "hq": hq,
                "hkv": hkv, "d": 128}
    if kind == "ffn":
        return {"kind": kind, "tokens": _log_int(rng, 1, 990), "hidden": hidden, "inter": inter}
    chunk = _log_int(rng, 2, 190) if rng.random() < 0.6 else 0
    return {"kind": "model", "layers": rng.choice([2, 3, 4]), "decodes": _log_int(rng, 1, 64),
            "median": _log_int(rng, 128, 1024), "longest": 4096, "chunk": chunk,
            "prior": _log_int(rng, 1, 2048) if chunk and rng.random() < 0.5 else 0,
            "rows_seed": rng.randrange(1 << 30)}


# ---------------------------------------------------------------- rows and work

def _contexts(n, median, longest, long_share, rng):
    x = np.clip(np.round(rng.lognormal(math.log(median), 1.0, n)), 1, longest).astype(np.int64)
    far = rng.integers(longest // 4, longest + 1, n)
    return np.where(rng.random(n) < long_share, far, x)


def _starts_lens(case):
    """(start, length) of every row: decode rows first, then the chunks."""
    rng = np.random.default_rng(case["rows_seed"])
    ctx = _contexts(case["decodes"], case["median"], case["longest"], case.get("long_share", 0.0),
                    rng)
    rows = [(int(c) - 1, 1) for c in ctx]
    if case["kind"] == "model":
        return rows + ([(case["prior"], case["chunk"])] if case["chunk"] else [])
    for c in case["chunks"].split():
        length, prior = c.split("@")
        rows.append((int(prior), int(length)))
    return rows


def _attention_work(rows, hq, hkv, d, block):
    tokens = sum(c for _, c in rows)
    flops = 4.0 * d * hq * sum(c * s + c * (c + 1) / 2 for s, c in rows)
    read = 4.0 * hkv * d * sum(s for s, _ in rows)        # prior K and V rows
    read += 4.0 * sum(-(-(s + c) // block) for s, c in rows)  # block tables
    return tokens, flops, read


def work(case):
    kind = case["kind"]
    if kind == "step":
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        tokens, flops, read = _attention_work(_starts_lens(case), hq, hkv, d, case["block"])
        # q read, out written; new K and V rows read and written to the pools
        return {"bytes": read + tokens * d * (4.0 * hq + 8.0 * hkv), "flops": flops}
    if kind == "attn_proj":
        t, h, hq, hkv, d = (case[k] for k in ("tokens", "hidden", "hq", "hkv", "d"))
        n = (hq + 2 * hkv) * d
        weights = n * h + h * hq * d + h + 2 * d
        # x, attn read; q, k, v and the sum written
        return {"bytes": 2.0 * (weights + t * (2 * h + hq * d + n)) + 4.0 * t,
                "flops": 2.0 * t * h * (n + hq * d)}
    if kind == "ffn":
        t, h, i = case["tokens"], case["hidden"], case["inter"]
        return {"bytes": 2.0 * (3 * h * i + h + 2 * t * h), "flops": 6.0 * t * h * i}
    c = M.QWEN3_8B
    rows = _starts_lens(case)
    tokens, flops, read = _attention_work(rows, c.hq, c.hkv, c.head_dim, c.block_size)
    layer = (2 * c.hq + 2 * c.hkv) * c.head_dim * c.hidden + 3 * c.hidden * c.inter
    per_layer = read + 4.0 * tokens * c.hkv * c.head_dim + 2.0 * layer
    head = 2.0 * c.vocab * c.hidden + 2.0 * len(rows) * c.vocab
    return {"bytes": case["layers"] * per_layer + head + 4.0 * tokens * c.hidden,
            "flops": case["layers"] * (flops + 2.0 * tokens * layer)
            + 2.0 * len(rows) * c.vocab * c.hidden}


# ---------------------------------------------------------------- inputs

def _randn(gen, *shape, scale=1.0):
    t = torch.randn(*shape, generator=gen, device=DEV, dtype=torch.bfloat16)
    return t.mul_(scale) if scale != 1.0 else t


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _prepare_step(case, seed):
    hq, hkv, d, block = (case[k] for k in ("hq", "hkv", "d", "block"))
    rows = _starts_lens(case)
    need = [-(-(s + c) // block) for s, c in rows]
    rng = np.random.default_rng(seed)
    pool, width = sum(need) + 2, max(need)
    perm = rng.permutation(pool).astype(np.int32)
    slots = rng.permutation(len(rows))                     # each row's place in the table
    table = np.full((len(rows), width), perm[-1], np.int32)
    meta = np.zeros((len(rows), 4), np.int32)
    at = 0
    for i, (s, c) in enumerate(rows):
        table[slots[i], :need[i]] = perm[at:at + need[i]]
        at += need[i]
        meta[i] = (slots[i], s, c, s + c)
    g, t = _gen(seed), sum(c for _, c in rows)
    desc = cp.make_desc(hq, hkv, d, block, pool, width, len(rows), 1.0 / math.sqrt(d))
    return {"case": case, "desc": desc, "rows": meta, "table_host": table,
            "table": torch.from_numpy(table).to(DEV),
            "q": _randn(g, t, hq, d), "k_new": _randn(g, t, hkv, d), "v_new": _randn(g, t, hkv, d),
            "kc": _randn(g, pool, hkv, block, d), "vc": _randn(g, pool, hkv, d, block),
            "out": torch.empty(t, hq, d, dtype=torch.bfloat16, device=DEV),
            "ws": torch.empty(cp.workspace_bytes(desc, meta), dtype=torch.uint8, device=DEV)}


def _prepare_proj(case, seed):
    t, h, hq, hkv, d = (case[k] for k in ("tokens", "hidden", "hq", "hkv", "d"))
    g, n = _gen(seed), (hq + 2 * hkv) * d

    def empty(*shape):
        return torch.empty(*shape, dtype=torch.bfloat16, device=DEV)

    need = max(M.gemm_workspace_bytes(t, n, h), M.gemm_workspace_bytes(t, h, hq * d), 256)
    return {"case": case, "x": _randn(g, t, h), "attn": _randn(g, t, hq * d),
            "norm": _randn(g, h, scale=0.1).add_(1.0), "q_norm": _randn(g, d, scale=0.1).add_(1.0),
            "k_norm": _randn(g, d, scale=0.1).add_(1.0), "wqkv": _randn(g, n, h, scale=0.02),
            "wo": _randn(g, h, hq * d, scale=0.02),
            "pos": torch.randint(0, 32768, (t,), generator=g, device=DEV, dtype=torch.int32),
            "h": empty(t, h), "qkv": empty(t, n), "q": empty(t, hq, d), "k": empty(t, hkv, d),
            "v": empty(t, hkv, d), "y": empty(t, h),
            "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}


def _prepare_ffn(case, seed):
    t, h, i = case["tokens"], case["hidden"], case["inter"]
    g = _gen(seed)

    def empty(*shape):
        return torch.empty(*shape, dtype=torch.bfloat16, device=DEV)

    return {"case": case, "x": _randn(g, t, h), "norm": _randn(g, h, scale=0.1).add_(1.0),
            "gate_up": _randn(g, 2 * i, h, scale=0.02), "down": _randn(g, h, i, scale=0.02),
            "h": empty(t, h), "gu": empty(t, 2 * i), "act": empty(t, i), "y": empty(t, h)}


def _prepare_model(case, seed):
    starts = _starts_lens(case)
    rows = np.array([(i, s, c, s + c) for i, (s, c) in enumerate(starts)], np.int32)
    tokens = int(rows[:, 2].sum())
    longest = max(2048, -(-int(rows[:, 3].max()) // 16) * 16)
    cfg = M.ModelConfig(layers=case["layers"])
    m = M.Model(cfg, max_seqs=len(rows), max_seq_len=longest, max_tokens=tokens, seed=seed,
                lm_head=False, fill_caches=True)
    g = _gen(seed + 1)
    last = torch.from_numpy(np.cumsum(rows[:, 2]).astype(np.int64) - 1).to(DEV)
    n = len(rows)
    return {"case": case, "model": m, "rows": rows, "last": last,
            "lm_head": _randn(g, cfg.vocab, cfg.hidden, scale=0.02),
            "hl": torch.empty(n, cfg.hidden, dtype=torch.bfloat16, device=DEV),
            "logits": torch.empty(n, cfg.vocab, dtype=torch.bfloat16, device=DEV)}


def prepare(case, seed):
    return {"step": _prepare_step, "attn_proj": _prepare_proj, "ffn": _prepare_ffn,
            "model": _prepare_model}[case["kind"]](case, seed)


# ---------------------------------------------------------------- one pass

def run(s):
    case = s["case"]
    if case["kind"] == "step":
        cp.step_mixed(s["desc"], s["q"], s["k_new"], s["v_new"], s["kc"], s["vc"], s["table"],
                      s["rows"], s["out"], s["ws"])
        return {"out": s["out"], "k_cache": s["kc"], "v_cache": s["vc"]}
    if case["kind"] == "attn_proj":
        M.rmsnorm(s["x"], s["norm"], s["h"], EPS)
        M.project_attn(s["h"], s["wqkv"], s["qkv"], ws=s["ws"])
        M.qkv_rope(s["qkv"], s["q_norm"], s["k_norm"], s["pos"], case["hq"], case["hkv"],
                   case["d"], THETA, EPS, s["q"], s["k"], s["v"])
        M.project_attn(s["attn"], s["wo"], s["y"], residual=s["x"], ws=s["ws"])
        return {"q": s["q"], "k": s["k"], "v": s["v"], "y": s["y"]}
    if case["kind"] == "ffn":
        M.rmsnorm(s["x"], s["norm"], s["h"], EPS)
        M.project(s["h"], s["gate_up"], s["gu"])
        M.swiglu(s["gu"], s["act"])
        M.project(s["act"], s["down"], s["y"], residual=s["x"])
        return {"y": s["y"]}
    m = s["model"]
    m.forward(s["rows"])
    x = m.x[:int(s["rows"][:, 2].sum())]
    M.rmsnorm(x.index_select(0, s["last"]), m.final_norm, s["hl"], EPS)
    M.project(s["hl"], s["lm_head"], s["logits"])
    return {"logits": s["logits"], "hidden": x}


# ---------------------------------------------------------------- 64-bit results

def _norm64(x, w):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * w.double()


def _rope64(x, pos):
    """x [T, heads, D]; elements d and d + D/2 turn by pos * THETA^(-2d/D)."""
    half = x.shape[-1] // 2
    f = THETA ** (-torch.arange(half, device=DEV, dtype=torch.float64) * 2 / x.shape[-1])
    a = pos.double()[:, None, None] * f
    c, s, lo, hi = a.cos(), a.sin(), x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _qkv64(qkv, q_norm, k_norm, pos, hq, hkv, d):
    x = qkv.view(-1, hq + 2 * hkv, d)
    q, k, v = x.split([hq, hkv, hkv], 1)
    return _rope64(_norm64(q, q_norm), pos), _rope64(_norm64(k, k_norm), pos), v


def _swiglu64(gu):
    g, u = gu.chunk(2, -1)
    return g / (1 + torch.exp(-g)) * u


def _mm64(a, w):
    return a @ w.double().t()


def _attend64(q, k, v, start, scale):
    """q [c, hq, d] at positions start.. over k, v [hkv, ctx, d]."""
    c, hq, d = q.shape
    hkv, ctx, _ = k.shape
    g = hq // hkv
    out = torch.empty(c, hq, d, dtype=torch.float64, device=DEV)
    hidden = (torch.arange(ctx, device=DEV)[None, :]
              > (start + torch.arange(c, device=DEV))[:, None]) if c > 1 else None
    for h in range(hkv):
        for first in range(0, c, 512):
            part = q[first:first + 512, h * g:(h + 1) * g].reshape(-1, d)
            s = (part @ k[h].t()).mul_(scale).view(-1, g, ctx)
            if hidden is not None:
                s.masked_fill_(hidden[first:first + 512, None, :], -math.inf)
            w = torch.softmax(s, -1).view(-1, ctx)
            out[first:first + 512, h * g:(h + 1) * g] = (w @ v[h]).view(-1, g, d)
    return out


def _place(kc, vc, blocks, start, k, v):
    """Rows k, v [c, hkv, d] written at positions start.. of one request's pages."""
    block = kc.shape[2]
    p = torch.arange(start, start + k.shape[0], device=DEV)
    b, o = blocks[p // block].long(), p % block
    kc[b, :, o, :] = k.to(kc.dtype)
    vc[b, :, :, o] = v.to(vc.dtype)


def _pages64(kc, vc, blocks, ctx):
    block = kc.shape[2]
    b = blocks[:-(-ctx // block)].long()
    k = kc[b].double().permute(1, 0, 2, 3).reshape(kc.shape[1], -1, kc.shape[3])
    v = vc[b].double().permute(1, 0, 3, 2).reshape(kc.shape[1], -1, kc.shape[3])
    return k[:, :ctx].contiguous(), v[:, :ctx].contiguous()


def _exact_step(case, s):
    out = torch.empty(s["out"].shape, dtype=torch.float64, device=DEV)
    scale, at, q = float(s["desc"].sm_scale), 0, s["q"].double()
    for slot, start, c, ctx in s["rows"].tolist():
        blocks = s["table"][slot]
        _place(s["kc"], s["vc"], blocks, start, s["k_new"][at:at + c], s["v_new"][at:at + c])
        k, v = _pages64(s["kc"], s["vc"], blocks, ctx)
        out[at:at + c] = _attend64(q[at:at + c], k, v, start, scale)
        at += c
    return {"out": out, "k_cache": s["kc"], "v_cache": s["vc"]}


def _exact_model(case, s):
    m, rows = s["model"], s["rows"].tolist()
    cfg, t = m.cfg, int(s["rows"][:, 2].sum())
    x = m.embed[m.tokens[:t]].double()
    pos = torch.cat([torch.arange(a, a + c, device=DEV) for _, a, c, _ in rows])
    for w, kc, vc in zip(m.layers, m.kc, m.vc):
        q, k, v = _qkv64(_mm64(_norm64(x, w["in_norm"]), w["qkv"]), w["q_norm"], w["k_norm"], pos,
                         cfg.hq, cfg.hkv, cfg.head_dim)
        o, at = torch.empty_like(q), 0
        for slot, start, c, ctx in rows:
            kp, vp = _pages64(kc, vc, m.bt[slot], ctx)
            kp[:, start:ctx] = k[at:at + c].transpose(0, 1)   # the new rows, unrounded
            vp[:, start:ctx] = v[at:at + c].transpose(0, 1)
            o[at:at + c] = _attend64(q[at:at + c], kp, vp, start, 1.0 / math.sqrt(cfg.head_dim))
            at += c
        x = x + _mm64(o.reshape(t, -1), w["o"])
        x = x + _mm64(_swiglu64(_mm64(_norm64(x, w["post_norm"]), w["gate_up"])), w["down"])
    logits = _mm64(_norm64(x[s["last"]], m.final_norm), s["lm_head"])
    return {"logits": logits, "hidden": x}


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "step":
        return _exact_step(case, s)
    if case["kind"] == "model":
        return _exact_model(case, s)
    x = s["x"].double()
    h = _norm64(x, s["norm"])
    if case["kind"] == "attn_proj":
        q, k, v = _qkv64(_mm64(h, s["wqkv"]), s["q_norm"], s["k_norm"], s["pos"], case["hq"],
                         case["hkv"], case["d"])
        return {"q": q, "k": k, "v": v, "y": x + _mm64(s["attn"].double(), s["wo"])}
    return {"y": x + _mm64(_swiglu64(_mm64(h, s["gate_up"])), s["down"])}


# ---------------------------------------------------------------- tolerances

# Relative errors against the 64-bit results: step 1.8e-3 to 2.3e-3, attn_proj
# 1.7e-3 to 2.9e-3, ffn 3.9e-3 (three roundings to bf16 in a row), model 1.4e-2
# (four layers of them); about four times that, at most 3e-2.
def tolerance(case):
    return {"rel": {"step": 8e-3, "attn_proj": 1.1e-2, "ffn": 1.5e-2, "model": 3e-2}[case["kind"]]}
