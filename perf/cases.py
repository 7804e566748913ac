"""The calls a user of the verification library makes, as timed cases.

Every case goes through the methods of `flexverify.Context`, on inputs that are already on the GPU (a serving program has
its weights re-tiled, its sessions in pages and the received drafts uploaded before it calls).  Inputs come from the seed
alone; the recipes are those of `synth` (weights N(0, 0.02), cached K / V N(0, 1), ragged contexts and draft lengths),
except that the draft laws do not depend on the library's own logits: they are softmaxes of independent N(0, 2) rows, from
which the drafts are drawn.  About a quarter of the drafts is accepted at the model calls.

What a model call returns here is its logits and the KV pools it appended to.  The accepted lengths and tokens of the bf16
model calls are left out: with a nearly flat law over 10^5 ids the drawn id moves with any change of rounding.  The
decisions are compared as whole numbers where the logits are given (the sampling cases) and on the fp32 model.
"""
from __future__ import annotations

import dataclasses
import math
import random

import numpy as np
import torch

from paper_2601_00644_amd import flexverify as fv
from paper_2601_00644_amd import synth

DEV = "cuda"
HEAD_HIDDEN, HEAD_PROJ, HEAD_STD = 2048, 2048, 0.04      # head of the draft model (widths: multiples of 256)


def listed():
    return [
        # the fp32 decoder of the correctness configuration: one request, 128 cached positions, four drafts; the smallest call
        dict(name="verify_tiny_f32", kind="verify", model="tiny", layers=2, vocab=4096, batch=1, ctx_lo=128, ctx_hi=128,
             gamma_lo=4, gamma_hi=4, temperature=1.0, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0),
        # one user on a 1B target: latency of a single request's verification, the whole model
        dict(name="verify_1b_one", kind="verify", model="llama1b", layers=16, vocab=128256, batch=1, ctx_lo=2048, ctx_hi=2048,
             gamma_lo=4, gamma_hi=4, temperature=1.0, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0),
        # long sessions on the 1B target with long draft blocks (good links): attention over 10^4 positions, head size 64
        dict(name="verify_1b_long", kind="verify", model="llama1b", layers=16, vocab=128256, batch=8, ctx_lo=4096, ctx_hi=16384,
             gamma_lo=8, gamma_hi=16, temperature=1.0, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0),
        # the serving configuration: 16 requests on the 8B target, ragged contexts and drafts, the whole model
        dict(name="verify_8b_b16", kind="verify", model="llama8b", layers=32, vocab=128256, batch=16, ctx_lo=512, ctx_hi=4096,
             gamma_lo=1, gamma_hi=8, temperature=0.8, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0),
        # a full batch of 128 requests through four 8B layers (the 32-layer call repeats them; the vocabulary is cut with
        # them so that the head keeps about its share)
        dict(name="verify_8b4_b128", kind="verify", model="llama8b", layers=4, vocab=32000, batch=128, ctx_lo=256, ctx_hi=8192,
             gamma_lo=1, gamma_hi=12, temperature=1.0, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0),
        # evolved targets: requests of three adapters and of the base target in one batch, nucleus sampling, every fourth
        # request greedy; four 8B layers with the full vocabulary (the cut works on the head's fp32 logits)
        dict(name="verify_8b4_adapted", kind="verify", model="llama8b", layers=4, vocab=128256, batch=16, ctx_lo=512, ctx_hi=4096,
             gamma_lo=1, gamma_hi=8, temperature=0.8, greedy_every=4, top_p=0.9, top_k=0, adapters=3, rank=16),
        # restoring sessions from tokens: a new prompt and one that continues a cached context, 2048 rows in pieces of 16
        dict(name="prefill_8b4", kind="prefill", model="llama8b", layers=4, vocab=32000, ctx_a=0, rows_a=1401, ctx_b=2050,
             rows_b=647, piece=16),
        # accept / resample on given bf16 logits: 64 requests, up to 16 drafts, a large vocabulary
        dict(name="sample_bf16", kind="sample", dtype="bf16", batch=64, gamma_lo=1, gamma_hi=16, vocab=152064, temperature=0.7,
             greedy_every=0, top_p=1.0, top_k=0),
        # the same step on fp32 logits with the usual sampling cuts (top-k, then top-p)
        dict(name="sample_f32_cut", kind="sample", dtype="f32", batch=32, gamma_lo=1, gamma_hi=8, vocab=128256, temperature=0.8,
             greedy_every=0, top_p=0.9, top_k=50),
        # the draft laws recomputed on the cloud before a verification call (anchor block + head + softmax), 16 requests
        dict(name="draft_probs_8b", kind="draft", model="llama8b", layers=2, vocab=128256, batch=16, ctx_lo=512, ctx_hi=4096,
             gamma_lo=1, gamma_hi=8, temperature=0.8),
        # one user's session saved, another's restored (32 layers of the 8B KV geometry)
        dict(name="kv_swap_8b", kind="kv", model="llama8b", layers=32, pos_out=2777, pos_in=3100),
        # one layer's attention on its own, 16 ragged requests
        dict(name="attention_8b_b16", kind="attention", model="llama8b", batch=16, ctx_lo=512, ctx_hi=4096, gamma_lo=1, gamma_hi=8),
    ]


def draw(rng):
    """One more case of the same ranges; none costs more than the 32-layer call of 16 requests."""
    def logi(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["verify", "verify", "verify", "prefill", "sample", "sample", "draft", "kv", "attention"])
    cut = dict(top_p=rng.choice([1.0, 1.0, 0.9, 0.95]), top_k=rng.choice([0, 0, 0, 50, 40]))
    lo = logi(100, 4000)
    ctx = dict(ctx_lo=lo, ctx_hi=logi(lo, 8192))
    g0 = rng.randint(1, 8)
    gam = dict(gamma_lo=g0, gamma_hi=rng.randint(g0, 16))
    T = rng.choice([0.6, 0.7, 0.8, 1.0])
    if kind == "verify":
        model = rng.choice(["tiny", "llama1b", "llama8b", "llama8b"])
        if model == "tiny":
            return dict(kind="verify", model="tiny", layers=2, vocab=4096, batch=1, ctx_lo=lo % 400 + 20, ctx_hi=lo % 400 + 20,
                        gamma_lo=g0, gamma_hi=g0, temperature=1.0, greedy_every=0, top_p=1.0, top_k=0, adapters=0, rank=0)
        batch = logi(1, 64)
        adapters = rng.choice([0, 0, 1, 2, 5]) if model == "llama8b" else 0
        return dict(kind="verify", model=model, layers=rng.randint(2, 4) if model == "llama8b" else rng.randint(4, 8),
                    vocab=rng.choice([32000, 128256, 50257]), batch=batch, **ctx, **gam, temperature=T,
                    greedy_every=rng.choice([0, 0, 2, 5]), **cut, adapters=adapters, rank=rng.choice([8, 16, 32]) if adapters else 0)
    if kind == "prefill":
        return dict(kind="prefill", model=rng.choice(["llama1b", "llama8b"]), layers=rng.randint(2, 4), vocab=32000,
                    ctx_a=rng.choice([0, logi(16, 2000)]), rows_a=logi(40, 1000), ctx_b=logi(100, 3000), rows_b=logi(40, 1000), piece=16)
    if kind == "sample":
        return dict(kind="sample", dtype=rng.choice(["bf16", "f32"]), batch=logi(1, 64), **gam,
                    vocab=rng.choice([32000, 50257, 128256, 152064, rng.randint(20000, 160000)]), temperature=T,
                    greedy_every=rng.choice([0, 0, 3]), **cut)
    if kind == "draft":
        return dict(kind="draft", model=rng.choice(["llama1b", "llama8b"]), layers=2, vocab=rng.choice([32000, 128256]),
                    batch=logi(1, 32), **ctx, **gam, temperature=T)
    if kind == "kv":
        return dict(kind="kv", model=rng.choice(["llama1b", "llama8b"]), layers=rng.randint(4, 32), pos_out=logi(50, 4000), pos_in=logi(50, 4000))
    return dict(kind="attention", model=rng.choice(["llama1b", "llama8b"]), batch=logi(1, 32), **ctx, **gam)


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed, stream, device=DEV):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 1000003 + 7919 * int(stream) + 11) & 0x7FFFFFFFFFFFFFFF)
    return g


def _cfg(case):
    cfg = synth.MODELS[case["model"]]
    kw = dict(n_layers=case.get("layers", 1), vocab=case.get("vocab", cfg.vocab))
    if case["kind"] in ("kv", "attention"):
        kw.update(d_ffn=256, vocab=256)     # neither call touches the MLP or the head
    return dataclasses.replace(cfg, **kw)


def _shape(case):
    """Context and draft lengths of the requests: part of the case, the same for every seed."""
    B = case["batch"]
    rng = random.Random(1000 * B + case["gamma_hi"] + case.get("ctx_hi", 0))
    L = [int(round(math.exp(rng.uniform(math.log(case["ctx_lo"]), math.log(case["ctx_hi"]))))) if case["ctx_hi"] > 8 * case["ctx_lo"]
         else rng.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(B)] if "ctx_lo" in case else [0] * B
    g = [rng.randint(case["gamma_lo"], case["gamma_hi"]) for _ in range(B)]
    return L, g


def _temps(case, B):
    t = np.full(B, case["temperature"], np.float32)
    if case.get("greedy_every"):
        t[case["greedy_every"] - 1::case["greedy_every"]] = 0.0
    return t


def _page_table(need, seed):
    """Physical pages of every session, scattered over the pool by a seeded permutation, none unused."""
    n, mp = sum(need), max(need)
    perm = np.random.default_rng(seed).permutation(n).astype(np.int32)
    pt, at = np.zeros((len(need), mp), np.int32), 0
    for b, k in enumerate(need):
        pt[b, :k] = perm[at:at + k]
        at += k
    return pt, n


def _context(cfg, L, seed, b, layers=None):
    """A session's cached K and V: [layers][L][kv heads][head_dim], N(0, 1)."""
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    shape = (cfg.n_layers if layers is None else layers, L, cfg.n_kv_heads, cfg.head_dim)
    return [torch.randn(shape, generator=_gen(seed, 1000 + 2 * b + i), device=DEV, dtype=torch.float32).to(dt) for i in (0, 1)]


def _laws(G, V, seed):
    """Draft laws [G][V] and the drafts drawn from them."""
    q = torch.randn((max(G, 1), V), generator=_gen(seed, 5), device=DEV, dtype=torch.float32).mul_(2.0).softmax(-1)
    d = _draw_rows(q, seed)
    return q, d


def _draw_rows(q, seed):
    u = torch.rand((q.shape[0], 1), generator=_gen(seed, 6), device=DEV, dtype=torch.float64)
    out = torch.empty(q.shape[0], dtype=torch.int32, device=DEV)
    for i in range(0, q.shape[0], 128):
        c = q[i:i + 128].double().cumsum(-1)
        out[i:i + 128] = torch.searchsorted(c, u[i:i + 128] * c[:, -1:]).clamp_(max=q.shape[1] - 1).squeeze(1).to(torch.int32)
    return out


def _tokens(V, n, seed, stream):
    return torch.randint(0, V, (n,), generator=_gen(seed, stream), device=DEV, dtype=torch.int32)


def _uniform(n, seed, stream):
    return torch.randint(0, 1 << 24, (max(n, 1),), generator=_gen(seed, stream), device=DEV).to(torch.float32) / float(1 << 24)


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def _cuts(case, batch, B):
    if case.get("top_p", 1.0) < 1.0:
        batch.top_p_host = np.full(B, case["top_p"], np.float32)
        batch.top_p = _dev(batch.top_p_host)
    if case.get("top_k", 0) > 0:
        batch.top_k_host = np.full(B, case["top_k"], np.int32)
        batch.top_k = _dev(batch.top_k_host)


def _adapters(case, cfg, seed):
    return [synth.make_lora(cfg, case["rank"], seed, a, device=DEV) for a in range(case["adapters"])]


def _sampled_logits(case, seed):
    V = case["vocab"]
    _, g = _shape(case)
    off = np.zeros(len(g) + 1, np.int32)
    off[1:] = np.cumsum(g)
    G, M = int(off[-1]), int(off[-1]) + len(g)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    logits = (torch.randn((M, V), generator=_gen(seed, 40), device=DEV) * 3.0).to(dt)
    rows = torch.as_tensor([int(off[b]) + b + i for b in range(len(g)) for i in range(g[b])], device=DEV)
    q = torch.empty((G, V), dtype=torch.float32, device=DEV)
    gen = _gen(seed, 41)
    for i in range(0, G, 64):       # the edge model's law: the target's with noise of 0.7 on the scaled logits
        z = logits[rows[i:i + 64]].float() / case["temperature"]
        q[i:i + 64] = (z + 0.7 * torch.randn(z.shape, generator=gen, device=DEV)).softmax(-1)
    return logits, q, _draw_rows(q, seed), off


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sample":
        logits, q, d, off = _sampled_logits(case, seed)
        B, G, V = case["batch"], int(off[-1]), case["vocab"]
        temps = _temps(case, B)
        cfg = synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16")
        ctx = fv.Context(cfg, None, B, 16, sampler_only=True)
        batch = fv.DeviceBatch(None, None, _dev(off), d, q, _uniform(G, seed, 7), _uniform(B, seed, 8), _dev(temps), None, None,
                               None, 0, None, off, temps)
        _cuts(case, batch, B)
        return dict(kind=kind, ctx=ctx, batch=batch, res=fv.DeviceResult.alloc(B), logits=logits)
    cfg = _cfg(case)
    w = synth.make_weights(cfg, seed, device=DEV)
    if kind == "kv":
        need = [(case["pos_out"] + 15) // 16, (case["pos_in"] + 15) // 16]
        pt, n = _page_table(need, seed)
        ctx = fv.Context(cfg, w, max_batch=1, max_gamma=1, max_pages_per_req=max(need))
        del w
        kp, vp = fv.alloc_pools(cfg, n)
        t = _dev(pt)
        out, inn = _context(cfg, case["pos_out"], seed, 0), _context(cfg, case["pos_in"], seed, 1)
        ctx.kv_import(kp, vp, n, t[0], 0, *out)
        return dict(kind=kind, ctx=ctx, kp=kp, vp=vp, n=n, rows=(t[0], t[1]), pos_out=case["pos_out"], k_in=inn[0], v_in=inn[1])
    if kind == "prefill":
        chunks = [(0, case["ctx_a"], _tokens(cfg.vocab, case["rows_a"], seed, 50).cpu().numpy()),
                  (1, case["ctx_b"], _tokens(cfg.vocab, case["rows_b"], seed, 51).cpu().numpy())]
        need = [(L0 + len(tk) + 15) // 16 for _, L0, tk in chunks]
        pt, n = _page_table(need, seed)
        pieces = sum((len(tk) + case["piece"] - 1) // case["piece"] for _, _, tk in chunks)
        ctx = fv.Context(cfg, w, max_batch=pieces, max_gamma=case["piece"] - 1, max_pages_per_req=max(need),
                         max_rows=case["rows_a"] + case["rows_b"])
        del w
        kp, vp = fv.alloc_pools(cfg, n)
        for s, L0, _ in chunks:
            if L0:
                ctx.kv_import(kp, vp, n, _dev(pt[s]), 0, *_context(cfg, L0, seed, s))
        return dict(kind=kind, ctx=ctx, batch=fv.prefill_pieces(chunks, pt, kp, vp, n, case["piece"]))
    # calls on a batch of requests
    L, g = _shape(case)
    B, V = case["batch"], cfg.vocab
    off = np.zeros(B + 1, np.int32)
    off[1:] = np.cumsum(g)
    G = int(off[-1])
    need = [(L[b] + g[b] + 1 + 15) // 16 for b in range(B)]
    pt, n = _page_table(need, seed)
    Lh = np.asarray(L, np.int32)
    ctx = fv.Context(cfg, w, max_batch=B, max_gamma=max(g), max_pages_per_req=max(need), max_rows=G + B)
    del w
    table = _dev(pt)
    one = kind == "draft"      # the draft model's session has one layer
    kp, vp = fv.alloc_draft_pools(cfg, n) if one else fv.alloc_pools(cfg, n)
    for b in range(B):
        k, v = _context(cfg, L[b], seed, b, 1 if one else None)
        if one:
            ctx.draft_kv_import(kp, vp, n, table[b], 0, k[0], v[0])
        else:
            ctx.kv_import(kp, vp, n, table[b], 0, k, v)
    if kind == "attention":
        q = torch.randn((G + B, cfg.n_heads, cfg.head_dim), generator=_gen(seed, 60), device=DEV).to(torch.bfloat16)
        batch = fv.DeviceBatch(_dev(Lh), None, _dev(off), None, None, None, None, None, table, kp, vp, n, Lh, off)
        return dict(kind=kind, ctx=ctx, batch=batch, q=q)
    temps = _temps(case, B)
    last = _tokens(V, B, seed, 4)
    if one:
        ctx.draft_attach(synth.make_draft_head(cfg, HEAD_HIDDEN, HEAD_PROJ, seed, device=DEV, std=HEAD_STD))
        batch = fv.DeviceBatch(_dev(Lh), last, _dev(off), _tokens(V, max(G, 1), seed, 61), None, None, None, _dev(temps), table, kp,
                               vp, n, Lh, off, temps)
        return dict(kind=kind, ctx=ctx, batch=batch)
    q, d = _laws(G, V, seed)
    batch = fv.DeviceBatch(_dev(Lh), last, _dev(off), d, q, _uniform(G, seed, 7), _uniform(B, seed, 8), _dev(temps), table, kp, vp, n,
                           Lh, off, temps)
    _cuts(case, batch, B)
    if case["adapters"]:
        ctx.lora_load(_adapters(case, cfg, seed))
        batch.adapter = _dev(_adapter_ids(case))
    return dict(kind=kind, ctx=ctx, batch=batch, res=fv.DeviceResult.alloc(B, G + B, V, want_logits=True), whole=cfg.dtype == "f32")


def _adapter_ids(case):
    return (np.arange(case["batch"]) % (case["adapters"] + 1) - 1).astype(np.int32)


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "verify":
        b, r = state["batch"], state["res"]
        ctx.verify(b, r)
        out = dict(logits=r.logits_out, k=b.k_pool, v=b.v_pool)
        if state["whole"]:
            out.update(accepted=r.accepted_len, token=r.next_token, length=r.new_seq_lens, released=r.pages_released, flags=r.flags)
        return out
    if kind == "prefill":
        b = state["batch"]
        return dict(logits=ctx.prefill(b, want_logits=True), k=b.k_pool, v=b.v_pool)
    if kind == "sample":
        r = state["res"]
        ctx.sample(state["logits"], state["batch"], r)
        return dict(accepted=r.accepted_len, token=r.next_token, flags=r.flags)
    if kind == "draft":
        b = state["batch"]
        q, _ = ctx.draft_probs(b)
        return dict(q=q, k=b.k_pool, v=b.v_pool)
    if kind == "attention":
        return dict(out=ctx.attention(0, state["q"], state["batch"]))
    k, v = ctx.kv_export(state["kp"], state["vp"], state["n"], state["rows"][0], 0, state["pos_out"])
    ctx.kv_import(state["kp"], state["vp"], state["n"], state["rows"][1], 0, state["k_in"], state["v_in"])
    return dict(saved_k=k, saved_v=v, k=state["kp"], v=state["vp"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------


def work(case):
    kind = case["kind"]
    if kind == "sample":
        V, B = case["vocab"], case["batch"]
        M = sum(_shape(case)[1]) + B
        el = 2 if case["dtype"] == "bf16" else 4
        # every logits row once, the draft law of the row the token is drawn from, one value per tested draft
        return {"bytes": M * V * el + B * V * 4, "flops": 4.0 * M * V}
    cfg = _cfg(case)
    el = 2 if cfg.dtype == "bf16" else 4
    d, F, V = cfg.d_model, cfg.d_ffn, cfg.vocab
    qd, qkv, kvrow = cfg.n_heads * cfg.head_dim, cfg.qkv_dim, 2 * cfg.n_kv_heads * cfg.head_dim * el
    layer = qkv * d + d * qd + 3 * F * d
    if kind == "kv":
        return {"bytes": 2.0 * cfg.n_layers * (case["pos_out"] + case["pos_in"]) * kvrow, "flops": 0.0}
    if kind == "prefill":
        M = case["rows_a"] + case["rows_b"]
        ctx = case["ctx_a"] + case["ctx_b"]
        pairs = sum(case["rows_" + s] * (case["ctx_" + s] + case["rows_" + s] / 2) for s in "ab")
        return {"bytes": el * (cfg.n_layers * layer + V * d + M * d) + cfg.n_layers * (ctx + M) * kvrow + 4.0 * M * V,
                "flops": 2.0 * M * (cfg.n_layers * layer + V * d) + cfg.n_layers * 4.0 * pairs * qd}
    L, g = _shape(case)
    tok, M = sum(L), sum(g) + len(g)
    pairs = sum(l * (x + 1) for l, x in zip(L, g))
    if kind == "attention":
        return {"bytes": (tok + M) * kvrow + M * qd * (2 + 4), "flops": 4.0 * pairs * qd}
    if kind == "draft":
        head = HEAD_HIDDEN * d + HEAD_HIDDEN * HEAD_PROJ + V * HEAD_PROJ
        return {"bytes": el * (layer + head + M * d) + (tok + 2 * M) * kvrow + 4.0 * (M - case["batch"]) * V,
                "flops": 2.0 * M * (layer + head) + 4.0 * pairs * qd}
    lora = case["adapters"] * case["rank"] * (2 * d + qd + qkv) * (cfg.n_layers - 1) if case["adapters"] else 0
    return {"bytes": el * (cfg.n_layers * layer + V * d + lora + M * d) + cfg.n_layers * (tok + 2 * M) * kvrow + 4.0 * M * V + 4.0 * case["batch"] * V,
            "flops": 2.0 * M * (cfg.n_layers * layer + V * d) + cfg.n_layers * 4.0 * pairs * qd}


def tolerance(case):
    kind = case["kind"]
    if kind in ("sample", "kv"):
        return "exact"                      # whole numbers; copies of bf16 values
    # about four times the distance from 64 bits measured on these inputs
    if kind == "attention":
        return {"rel": 1e-3}                # 2e-4: the fp16 output and the hi + lo pairs of the operands
    if kind == "verify" and case["model"] == "tiny":
        return {"rel": 2e-6}                # 3e-7: 32-bit sums
    if kind == "verify" and case["layers"] <= 8 and not case["adapters"]:
        return {"rel": 2e-2}                # 3 .. 5e-3: 16-bit tensors between the kernels of a few layers
    return {"rel": 3e-2}                    # 7e-3 .. 1.1e-2: 16 and 32 layers, adapters of unit size, short prompts, laws


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x: [rows][heads][hd]; pairs (i, i + hd/2)."""
    half = x.shape[-1] // 2
    f = theta ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / (2 * half))
    a = pos.double()[:, None, None] * f
    x0, x1 = x[..., :half], x[..., half:]
    return torch.cat([x0 * a.cos() - x1 * a.sin(), x0 * a.sin() + x1 * a.cos()], -1)


def _attend(q, k, v, L):
    """q: [n][H][hd] at positions L ..; k, v: [L + n][Hkv][hd]."""
    n, H, hd = q.shape
    grp = H // k.shape[1]
    out = torch.empty_like(q)
    mask = torch.arange(k.shape[0], device=DEV)[None, :] > (L + torch.arange(n, device=DEV))[:, None]
    for h in range(H):
        s = torch.mm(q[:, h], k[:, h // grp].t().contiguous()) / math.sqrt(hd)
        out[:, h] = torch.mm(s.masked_fill(mask, -math.inf).softmax(-1), v[:, h // grp].contiguous())
    return out


def _block(cfg, w, l, x, reqs, pos, cache, lora=None):
    """One decoder layer over the rows of all requests.  reqs: [(first row, rows, L)]; cache(b) -> the layer's K, V before
    the call; returns x and the appended K, V rows."""
    qd, kd = cfg.n_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim
    a = _norm(x, w[f"attn_norm.{l}"], cfg.rms_eps)
    qkv = a @ w[f"w_qkv.{l}"].double().t()
    for b, ad in lora or []:
        r0, n, _ = reqs[b]
        qkv[r0:r0 + n] += ad["scale"] * ((a[r0:r0 + n] @ ad["a_qkv"][l].double().t()) @ ad["b_qkv"][l].double().t())
    M = x.shape[0]
    q = _rope(qkv[:, :qd].reshape(M, cfg.n_heads, cfg.head_dim), pos, cfg.rope_theta)
    k = _rope(qkv[:, qd:qd + kd].reshape(M, cfg.n_kv_heads, cfg.head_dim), pos, cfg.rope_theta)
    v = qkv[:, qd + kd:].reshape(M, cfg.n_kv_heads, cfg.head_dim)
    att = torch.empty((M, qd), dtype=torch.float64, device=DEV)
    for b, (r0, n, L) in enumerate(reqs):
        ck, cv = cache(b)
        att[r0:r0 + n] = _attend(q[r0:r0 + n], torch.cat([ck.double(), k[r0:r0 + n]]), torch.cat([cv.double(), v[r0:r0 + n]]), L).reshape(n, qd)
    o = att @ w[f"w_o.{l}"].double().t()
    for b, ad in lora or []:
        r0, n, _ = reqs[b]
        o[r0:r0 + n] += ad["scale"] * ((att[r0:r0 + n] @ ad["a_o"][l].double().t()) @ ad["b_o"][l].double().t())
    x = x + o
    gu = _norm(x, w[f"mlp_norm.{l}"], cfg.rms_eps) @ w[f"w_gate_up.{l}"].double().t()
    g, u = gu[:, :cfg.d_ffn], gu[:, cfg.d_ffn:]
    return x + (g * torch.sigmoid(g) * u) @ w[f"w_down.{l}"].double().t(), k, v


def _pool64(cfg, n_pages, page_rows, seqs, layers):
    """The pools in 64 bits: seqs[b] = (K, V) [layers][positions][kv heads][hd]; the element order inside a page tile is the
    one the header documents for fsv_kv_import."""
    hd, H = cfg.head_dim, cfg.n_kv_heads
    t, e = torch.meshgrid(torch.arange(16, device=DEV), torch.arange(hd, device=DEV), indexing="ij")
    if cfg.dtype == "bf16":
        ko = ((e // 16 * 2 + (e % 16) // 8) * 16 + t) * 8 + e % 8
        vo = ((e // 32 * 2 + (t % 8) // 4) * 32 + e % 32) * 8 + 4 * (t // 8) + t % 4
    else:
        ko = vo = t * hd + e
    pools = []
    for which, order in ((0, ko), (1, vo)):
        inv = torch.empty(16 * hd, dtype=torch.long, device=DEV)
        inv[order.reshape(-1)] = torch.arange(16 * hd, device=DEV)
        pool = torch.zeros((layers, n_pages, H, 16 * hd), dtype=torch.float64, device=DEV)
        for b, s in enumerate(seqs):
            x = s[which]
            P = x.shape[1]
            np_ = (P + 15) // 16
            pages = torch.as_tensor(page_rows[b][:np_].astype(np.int64), device=DEV)
            for l in range(layers):
                y = torch.zeros((np_ * 16, H, hd), dtype=torch.float64, device=DEV)
                y[:P] = x[l]
                y = y.reshape(np_, 16, H, hd).permute(0, 2, 1, 3).reshape(np_, H, 16 * hd)
                pool[l, pages] = y[:, :, inv]
        pools.append(pool)
    return pools


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None                         # whole numbers
    cfg = _cfg(case)
    if kind == "kv":
        out, inn = _context(cfg, case["pos_out"], seed, 0), _context(cfg, case["pos_in"], seed, 1)
        pt, n = _page_table([(case["pos_out"] + 15) // 16, (case["pos_in"] + 15) // 16], seed)
        k, v = _pool64(cfg, n, pt, [out, inn], cfg.n_layers)
        return dict(saved_k=out[0].double(), saved_v=out[1].double(), k=k, v=v)
    if kind == "prefill":
        toks = [_tokens(cfg.vocab, case["rows_a"], seed, 50), _tokens(cfg.vocab, case["rows_b"], seed, 51)]
        L, rows = [case["ctx_a"], case["ctx_b"]], [case["rows_a"], case["rows_b"]]
    else:
        L, g = _shape(case)
        rows = [x + 1 for x in g]
        off = [0]
        for x in g:
            off.append(off[-1] + x)
        if kind != "attention":
            last, G = _tokens(cfg.vocab, case["batch"], seed, 4), off[-1]
            d = _tokens(cfg.vocab, max(G, 1), seed, 61) if kind == "draft" else _laws(G, cfg.vocab, seed)[1]
            toks = [torch.cat([last[b:b + 1], d[off[b]:off[b + 1]]]) for b in range(len(g))]
    first = [0]
    for x in rows:
        first.append(first[-1] + x)
    reqs = [(first[b], rows[b], L[b]) for b in range(len(L))]
    if kind == "attention":
        q = torch.randn((first[-1], cfg.n_heads, cfg.head_dim), generator=_gen(seed, 60), device=DEV).to(torch.bfloat16).double()
        out = torch.empty((first[-1], cfg.n_heads * cfg.head_dim), dtype=torch.float64, device=DEV)
        for b, (r0, n, Lb) in enumerate(reqs):
            k, v = (t[0].double() for t in _context(cfg, Lb, seed, b))
            pad = torch.zeros((n,) + tuple(k.shape[1:]), dtype=torch.float64, device=DEV)   # the call appends nothing: the slots are zero
            out[r0:r0 + n] = _attend(q[r0:r0 + n], torch.cat([k, pad]), torch.cat([v, pad]), Lb).reshape(n, -1)
        return dict(out=out)
    w = synth.make_weights(cfg, seed, device=DEV)
    pos = torch.cat([torch.arange(Lb, Lb + n, device=DEV) for _, n, Lb in reqs])
    x = w["embed"][torch.cat(toks).long()].double()
    one = kind == "draft"
    layers = 1 if one else cfg.n_layers
    ctxs = [_context(cfg, Lb, seed, b, layers) for b, (_, _, Lb) in enumerate(reqs)]
    new = []
    ads = _adapters(case, cfg, seed) if case.get("adapters") else []
    ids = _adapter_ids(case) if ads else []
    for j in range(layers):
        l = cfg.n_layers - 1 if one else j
        lora = [(b, ads[i]) for b, i in enumerate(ids) if i >= 0] if l < cfg.n_layers - 1 else None
        x, k, v = _block(cfg, w, l, x, reqs, pos, lambda b: (ctxs[b][0][j], ctxs[b][1][j]), lora)
        new.append((k, v))
    seqs = [[torch.cat([ctxs[b][i].double(), torch.stack([nk[i][r0:r0 + n] for nk in new])], 1) for i in (0, 1)]
            for b, (r0, n, _) in enumerate(reqs)]
    del ctxs
    pt, npg = _page_table([(Lb + n + 15) // 16 for _, n, Lb in reqs], seed)
    kp, vp = _pool64(cfg, npg, pt, seqs, layers)
    if one:
        h = synth.make_draft_head(cfg, HEAD_HIDDEN, HEAD_PROJ, seed, device=DEV, std=HEAD_STD)
        y = x @ h["w1"].double().t()
        z = ((y * torch.sigmoid(y)) @ h["w2"].double().t()) @ h["wv"].double().t()
        keep = torch.cat([torch.arange(r0, r0 + n - 1, device=DEV) for r0, n, _ in reqs])
        return dict(q=(z[keep] / float(np.float32(case["temperature"]))).softmax(-1), k=kp, v=vp)
    logits = _norm(x, w["final_norm"], cfg.rms_eps) @ w["lm_head"].double().t()
    out = dict(logits=logits, k=kp, v=vp)
    if cfg.dtype == "f32":
        out.update(accepted=None, token=None, length=None, released=None, flags=None)
    return out
