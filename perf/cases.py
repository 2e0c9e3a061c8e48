"""Timed cases of the library's use in serving: attention steps over the paged cache, the MLP's two
projections, and one decoder layer's library calls, at sizes from one decode row to a 16k-token chunk.

Shapes are those of the repository's workloads (paper_2608_15171_amd/inputs.py, layer_cost.py): 16 query and
2 KV heads of 128 features (or the two-way shard's 8 and 1), pages of 16 tokens, hidden 2048, 11008 intermediate
features (or the shard's 5504), contexts up to about 30k tokens.

A case is a step description (decode rows with contexts between ctx_lo and ctx_hi, then prefill chunks with
cached prefixes between cached_lo and cached_hi) or, for the MLP, a token count, plus the kind of call:
  attn    kv_append then attn_step: with a plan that the program keeps for the layers of an iteration
          ("planned"), or by the calls that plan for themselves ("direct")
  mlp     gateup_act then the down projection (gateup_proj)
  layer   the library's share of one decoder layer: Q, K and V projections, rotation and page write, attention,
          output projection, and the MLP's projections (the norms and residual adds are not the library's)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_15171_amd import ppas

PAGE, DIM, GROUP = 16, 128, 8
HIDDEN, THETA = 2048, 1e6
GOLDEN = 0.6180339887498949


def _step(kind, name, **kw):
    c = {"name": name, "kind": kind, "call": "planned", "kv_heads": 2, "decodes": 0, "ctx_lo": 0, "ctx_hi": 0,
         "chunks": 0, "chunk": 0, "cached_lo": 0, "cached_hi": 0}
    if kind == "layer":
        c["inter"] = 11008
    c.update(kw)
    return c


def _mlp(name, tokens, hidden=HIDDEN, inter=11008):
    return {"name": name, "kind": "mlp", "tokens": tokens, "hidden": hidden, "inter": inter}


def listed():
    return [
        # one user's decode step: the smallest call, launches and latencies
        _step("attn", "attn-decode-1", decodes=1, ctx_lo=3071, ctx_hi=3071),
        # a short prompt arriving while four requests decode, by the calls that plan for themselves
        _step("attn", "attn-mixed-512", call="direct", decodes=4, ctx_lo=1024, ctx_hi=1024, chunks=1, chunk=512),
        # many long-context requests decoding, no prefill in flight: the KV cache is streamed once
        _step("attn", "attn-decode-48", decodes=48, ctx_lo=20000, ctx_hi=30064),
        # a 2,048-token budget: one chunk late in a 25,000-token prompt beside eight decode rows
        _step("attn", "attn-chunk-2048", decodes=8, ctx_lo=25000, ctx_hi=25032, chunks=1, chunk=2048, cached_lo=22528,
              cached_hi=22528),
        # the 2,048-token budget under pressure: two chunks and 48 decode rows in one step
        _step("attn", "attn-pressure", decodes=48, ctx_lo=20000, ctx_hi=30064, chunks=2, chunk=1024, cached_lo=4926,
              cached_hi=12152),
        # the 16,384-token budget of a lightly loaded server: the last chunk of a 25,000-token prompt
        _step("attn", "attn-chunk-16384", chunks=1, chunk=16384, cached_lo=8616, cached_hi=8616),
        # the MLP of a decode iteration: the weights are streamed for a few rows
        _mlp("mlp-24", 24),
        # the MLP of a ragged prompt tail
        _mlp("mlp-700", 700),
        # the MLP of a 2,048-token chunk with eight decode rows
        _mlp("mlp-2056", 2056),
        # the MLP of a 16,384-token chunk
        _mlp("mlp-16384", 16384),
        # one layer of a decode iteration of 32 requests with ordinary contexts
        _step("layer", "layer-decode-32", decodes=32, ctx_lo=500, ctx_hi=4000),
        # one layer of an iteration that mixes a 1,000-token chunk and six decode rows
        _step("layer", "layer-chunk-1000", decodes=6, ctx_lo=2000, ctx_hi=9000, chunks=1, chunk=1000, cached_lo=3000,
              cached_hi=3000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges, never more work than the largest listed ones."""
    limit = {"attn": 2.2e12, "mlp": 2.2e12, "layer": 0.5e12}
    while True:
        kind = rng.choice(("attn", "attn", "mlp", "layer"))
        if kind == "mlp":
            c = _mlp("", _log(rng, 1, 16384), rng.choice((2048, 2048, 64 * rng.randint(8, 56))),
                     rng.choice((11008, 5504, rng.randint(500, 11008))))
            # the down projection reduces over the intermediate features: a multiple of 64
            c["inter"] = max(64, c["inter"] // 64 * 64)
        else:
            c = _step(kind, "", kv_heads=rng.choice((2, 2, 1)))
            if kind == "attn":
                c["call"] = rng.choice(("planned", "planned", "direct"))
            else:
                c["inter"] = 11008 if c["kv_heads"] == 2 else 5504
            shape = rng.choice(("decode", "chunk", "mixed"))
            if shape != "chunk":
                c["decodes"] = _log(rng, 1, 64)
                c["ctx_hi"] = _log(rng, 64, 30000)
                c["ctx_lo"] = rng.randint(c["ctx_hi"] // 4, c["ctx_hi"])
            if shape != "decode":
                c["chunks"] = rng.choice((1, 1, 2, 3))
                c["chunk"] = _log(rng, 9, 16384 if kind == "attn" else 4096)
                c["cached_hi"] = rng.choice((0, rng.randint(1, 25000)))
                c["cached_lo"] = rng.randint(0, c["cached_hi"])
        del c["name"]
        if work(c)["flops"] <= limit[kind] and work(c)["bytes"] <= 1.3e9:
            return c


# ---------------------------------------------------------------------------
# What a step's sizes come to
# ---------------------------------------------------------------------------

def _seqs(case):
    """(new tokens, cached tokens) of each request: decode rows first, then chunks."""
    def spread(lo, hi, i, n):
        return hi if n == 1 else lo + int((hi - lo) * ((i * GOLDEN) % 1.0))
    n, m = case["decodes"], case["chunks"]
    out = [(1, spread(case["ctx_lo"], case["ctx_hi"], i, n)) for i in range(n)]
    return out + [(case["chunk"], spread(case["cached_lo"], case["cached_hi"], i, m)) for i in range(m)]


def _attn_work(case):
    g = case["kv_heads"]
    seqs = _seqs(case)
    rows = sum(n for n, _ in seqs)
    keys = sum(n + c for n, c in seqs)
    pairs = sum(n * c + n * (n + 1) // 2 for n, c in seqs)
    # 4 x 128 per visible pair and query head; K and V of every visible token, Q and the output of every row, and
    # the new rows' K and V read once and written once
    return {"flops": 4.0 * DIM * GROUP * g * pairs,
            "bytes": float(keys * g * 512 + rows * GROUP * g * 512 + 2 * rows * g * 512)}


def _proj_work(t, k, n_in, n_out):
    return {"flops": 2.0 * t * k * n_in, "bytes": 2.0 * (t * k + n_in * k + t * n_out)}


def _sum(parts):
    return {m: sum(p[m] for p in parts) for m in ("flops", "bytes")}


def _mlp_work(t, hidden, inter):
    return _sum([_proj_work(t, hidden, 2 * inter, inter), _proj_work(t, inter, hidden, hidden)])


def work(case):
    if case["kind"] == "attn":
        return _attn_work(case)
    if case["kind"] == "mlp":
        return _mlp_work(case["tokens"], case["hidden"], case["inter"])
    t = sum(n for n, _ in _seqs(case))
    hq, hkv = GROUP * case["kv_heads"] * DIM, case["kv_heads"] * DIM
    return _sum([_attn_work(case), _mlp_work(t, HIDDEN, case["inter"]), _proj_work(t, HIDDEN, hq, hq),
                 _proj_work(t, HIDDEN, hkv, hkv), _proj_work(t, HIDDEN, hkv, hkv), _proj_work(t, hq, HIDDEN, HIDDEN)])


def tolerance(case):
    # Four times the error measured against 64 bits over the listed and two dozen drawn cases. Relative: attention
    # 2.4e-3 (probabilities and outputs rounded to bf16), the MLP 2.35e-3 (two roundings), a layer 3.8e-3 (the
    # rotated queries are rounded too). Largest single value: attention 4.6e-2 (first rows of a prompt, which see
    # few keys and are far larger than the output's root mean square), the MLP 1.2e-2, a layer 4.5e-2.
    return {"attn": {"rel": 0.0095, "max": 0.19}, "mlp": {"rel": 0.0095, "max": 0.05},
            "layer": {"rel": 0.015, "max": 0.18}}[case["kind"]]


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _rand(g, *shape, scale=1.0):
    """Normal values rounded to bf16: hidden states, queries, keys and values after normalisation, or weights."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    return out.normal_(0.0, scale, generator=g)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["kind"] == "mlp":
        t, h, i = case["tokens"], case["hidden"], case["inter"]
        s = {"case": case, "x": _rand(g, t, h), "gate_up": _rand(g, 2 * i, h, scale=0.02),
             "down": _rand(g, h, i, scale=0.02)}
        _mlp_buffers(s, t, h, i)
        return s
    seqs, hkv = _seqs(case), case["kv_heads"]
    rows = sum(n for n, _ in seqs)
    desc = np.zeros((len(seqs), 3), dtype=np.int32)
    at = 0
    for k, (n, c) in enumerate(seqs):
        desc[k] = (at, n, c)
        at += n
    need = [(n + c + PAGE - 1) // PAGE for n, c in seqs]
    pages = sum(need)
    order = np.random.Generator(np.random.PCG64(seed)).permutation(pages).astype(np.int32)
    bt = np.full((len(seqs), max(need)), -1, dtype=np.int32)
    at = 0
    for k, n in enumerate(need):
        bt[k, :n] = order[at:at + n]
        at += n
    s = {"case": case, "desc": desc, "bt_host": bt, "bt": torch.from_numpy(bt).cuda(),
         "shape": ppas.make_shape(GROUP * hkv, hkv, pages),
         "k_pages": _rand(g, pages, hkv, DIM // 8, PAGE, 8), "v_pages": _rand(g, pages, hkv, DIM, PAGE)}
    s["out"] = torch.empty((rows, GROUP * hkv, DIM), dtype=torch.bfloat16, device="cuda")
    if case["call"] == "planned":
        s["plan"] = ppas.StepPlan(s["shape"], desc, bt)
        nbytes = s["plan"].workspace_bytes
    else:
        nbytes = ppas.attn_workspace_bytes(s["shape"], desc)
    s["workspace"] = torch.empty(max(256, nbytes), dtype=torch.uint8, device="cuda")
    if case["kind"] == "attn":
        s["q"] = _rand(g, rows, GROUP * hkv, DIM)
        s["k_new"], s["v_new"] = _rand(g, rows, hkv, DIM), _rand(g, rows, hkv, DIM)
        return s
    i = case["inter"]
    s["q"] = torch.empty((rows, GROUP * hkv, DIM), dtype=torch.bfloat16, device="cuda")
    s["k_new"] = torch.empty((rows, hkv, DIM), dtype=torch.bfloat16, device="cuda")
    s["v_new"] = torch.empty_like(s["k_new"])
    s["o"] = torch.empty((rows, HIDDEN), dtype=torch.bfloat16, device="cuda")
    s["x"] = _rand(g, rows, HIDDEN)
    for name, n, k in (("wq", GROUP * hkv * DIM, HIDDEN), ("wk", hkv * DIM, HIDDEN), ("wv", hkv * DIM, HIDDEN),
                       ("wo", HIDDEN, GROUP * hkv * DIM), ("gate_up", 2 * i, HIDDEN), ("down", HIDDEN, i)):
        s[name] = _rand(g, n, k, scale=0.02)
    _mlp_buffers(s, rows, HIDDEN, i,
                 max(ppas.gateup_workspace_bytes(rows, HIDDEN, GROUP * hkv * DIM),
                     ppas.gateup_workspace_bytes(rows, HIDDEN, hkv * DIM),
                     ppas.gateup_workspace_bytes(rows, GROUP * hkv * DIM, HIDDEN)))
    return s


def _mlp_buffers(s, t, h, i, least=0):
    s["z"] = torch.empty((t, i), dtype=torch.bfloat16, device="cuda")
    s["y"] = torch.empty((t, h), dtype=torch.bfloat16, device="cuda")
    nbytes = max(256, least, ppas.gateup_act_workspace_bytes(t, h, i), ppas.gateup_workspace_bytes(t, i, h))
    s["proj_ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    kind = s["case"]["kind"]
    if kind == "mlp":
        ppas.gateup_act(s["x"], s["gate_up"], s["z"], s["proj_ws"])
        ppas.gateup_proj(s["z"], s["down"], s["y"], s["proj_ws"])
        return {"z": s["z"], "y": s["y"]}
    pools = s["k_pages"], s["v_pages"]
    if kind == "attn":
        if s["case"]["call"] == "planned":
            s["plan"].kv_append(*pools, s["k_new"], s["v_new"], s["bt"])
            s["plan"].attn_step(s["out"], s["q"], *pools, s["bt"], s["workspace"])
        else:
            ppas.kv_append(s["shape"], *pools, s["k_new"], s["v_new"], s["desc"], s["bt"], s["bt_host"])
            ppas.attn_step(s["shape"], s["out"], s["q"], *pools, s["desc"], s["bt"], s["workspace"], s["bt_host"])
        return {"out": s["out"], "k_pages": s["k_pages"], "v_pages": s["v_pages"]}
    t = s["x"].shape[0]
    ppas.gateup_proj(s["x"], s["wq"], s["q"].view(t, -1), s["proj_ws"])
    ppas.gateup_proj(s["x"], s["wk"], s["k_new"].view(t, -1), s["proj_ws"])
    ppas.gateup_proj(s["x"], s["wv"], s["v_new"].view(t, -1), s["proj_ws"])
    s["plan"].rope_kv_append(THETA, s["q"], *pools, s["k_new"], s["v_new"], s["bt"])
    s["plan"].attn_step(s["out"], s["q"], *pools, s["bt"], s["workspace"])
    ppas.gateup_proj(s["out"].view(t, -1), s["wo"], s["o"], s["proj_ws"])
    ppas.gateup_act(s["x"], s["gate_up"], s["z"], s["proj_ws"])
    ppas.gateup_proj(s["z"], s["down"], s["y"], s["proj_ws"])
    return {"q": s["q"], "out": s["out"], "o": s["o"], "y": s["y"], "k_pages": s["k_pages"], "v_pages": s["v_pages"]}


# ---------------------------------------------------------------------------
# The same in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _mm(x, w):
    """x w^T in 64 bits, a few thousand rows at a time."""
    w = w.double()
    return torch.cat([x[r:r + 4096].double() @ w.t() for r in range(0, x.shape[0], 4096)])


def _mlp_exact(x, gate_up, down):
    i = gate_up.shape[0] // 2
    z, y = [], []
    for r in range(0, x.shape[0], 2048):
        a = _mm(x[r:r + 2048], gate_up)
        a = torch.nn.functional.silu(a[:, :i]) * a[:, i:]
        z.append(a)
        y.append(_mm(a, down))
    return torch.cat(z), torch.cat(y)


def _rotate(x, pos):
    """Rotate-half embedding of [rows, heads, 128] at the rows' positions."""
    half = DIM // 2
    inv = THETA ** (-torch.arange(half, device=x.device, dtype=torch.float64) * 2.0 / DIM)
    a = pos.double()[:, None, None] * inv
    c, n = a.cos(), a.sin()
    return torch.cat([x[..., :half] * c - x[..., half:] * n, x[..., half:] * c + x[..., :half] * n], dim=-1)


def _attend(s, q, k_new, v_new):
    """The attention of the step's rows: cached keys from the pools, the new ones as given (all 64-bit)."""
    hkv, outs = s["case"]["kv_heads"], []
    for k, (at, n, c) in enumerate(s["desc"].tolist()):
        ids = s["bt"][k, :(n + c + PAGE - 1) // PAGE].long()
        for g in range(hkv):
            kk = s["k_pages"][ids, g].permute(0, 2, 1, 3).reshape(-1, DIM)[:c].double()
            vv = s["v_pages"][ids, g].permute(0, 2, 1).reshape(-1, DIM)[:c].double()
            kk = torch.cat([kk, k_new[at:at + n, g]])
            vv = torch.cat([vv, v_new[at:at + n, g]])
            for r in range(0, n, 256):
                m = min(256, n - r)
                qq = q[at + r:at + r + m, GROUP * g:GROUP * (g + 1)].reshape(-1, DIM)
                logits = (qq @ kk[:c + r + m].t()).view(m, GROUP, -1) / math.sqrt(DIM)
                tail = logits[..., c + r:]
                hidden = torch.ones(m, m, dtype=torch.bool, device=q.device).triu(1)
                tail.masked_fill_(hidden[:, None, :], -math.inf)
                o = logits.softmax(-1).view(m * GROUP, -1) @ vv[:c + r + m]
                outs.append((at + r, m, g, o.view(m, GROUP, DIM)))
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for at, m, g, o in outs:
        out[at:at + m, GROUP * g:GROUP * (g + 1)] = o
    return out


def _appended(s, k_new, v_new):
    """The pools with the step's new rows written to their slots."""
    kp, vp = s["k_pages"].clone(), s["v_pages"].clone()
    for k, (at, n, c) in enumerate(s["desc"].tolist()):
        pos = torch.arange(c, c + n, device=kp.device)
        page, slot = s["bt"][k].long()[pos // PAGE], pos % PAGE
        hkv = kp.shape[1]
        kp[page, :, :, slot, :] = k_new[at:at + n].reshape(n, hkv, DIM // 8, 8).to(kp.dtype)
        vp[page, :, :, slot] = v_new[at:at + n].to(vp.dtype)
    return kp, vp


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "mlp":
        z, y = _mlp_exact(s["x"], s["gate_up"], s["down"])
        return {"z": z, "y": y}
    if case["kind"] == "attn":
        out = _attend(s, s["q"].double(), s["k_new"].double(), s["v_new"].double())
        kp, vp = _appended(s, s["k_new"], s["v_new"])
        return {"out": out, "k_pages": kp, "v_pages": vp}
    t, hkv = s["x"].shape[0], case["kv_heads"]
    pos = torch.cat([torch.arange(c, c + n, device="cuda") for _, n, c in s["desc"].tolist()])
    q = _rotate(_mm(s["x"], s["wq"]).view(t, -1, DIM), pos)
    k = _rotate(_mm(s["x"], s["wk"]).view(t, hkv, DIM), pos)
    v = _mm(s["x"], s["wv"]).view(t, hkv, DIM)
    out = _attend(s, q, k, v)
    kp, vp = _appended(s, k, v)
    return {"q": q, "out": out, "o": _mm(out.view(t, -1), s["wo"]), "y": _mlp_exact(s["x"], s["gate_up"], s["down"])[1],
            "k_pages": kp, "v_pages": vp}
