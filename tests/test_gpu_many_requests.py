"""Calls of thousands of requests: the set-up launch scans the requests in rounds of 1024 and keeps their prefix sums in LDS up
to 2048 of them, in memory beyond.  Every request has to get the rows, positions, tokens, parts and pages it gets in a small
batch, where both are one round."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1023, 1024, 1025, 2047, 2048, 2049, 3000])
def test_requests_get_what_they_get_in_small_batches(B):
    from paper_2601_00644_amd import flexverify as fv
    cfg = dataclasses.replace(synth.MODELS["mini64"], n_layers=1)
    rng = np.random.default_rng(B)
    gam = rng.integers(0, 2, B).astype(np.int32)
    L = rng.integers(0, 100, B).astype(np.int32)
    L[rng.permutation(B)[:24]] = rng.integers(900, 2000, 24)      # long enough for several parts in any batch
    L[B - 1] = 1500
    need = (L + gam + 16) // 16
    pt = np.zeros((B, int(need.max())), np.int32)
    n = int(need.sum())
    perm = rng.permutation(n).astype(np.int32)
    at = np.concatenate([[0], np.cumsum(need)])
    for b in range(B):
        pt[b, :need[b]] = perm[at[b]:at[b + 1]]
    g = torch.Generator().manual_seed(B)
    w = {k: v.cuda() for k, v in synth.make_weights(cfg, 2, std=0.05).items()}
    ctx = fv.Context(cfg, w, max_batch=B, max_gamma=1, max_pages_per_req=pt.shape[1], max_rows=2 * B)
    kp, vp = fv.alloc_pools(cfg, n)
    kp.copy_(torch.randn(kp.shape, generator=g).to(kp.dtype))
    vp.copy_(torch.randn(vp.shape, generator=g).to(vp.dtype))
    last, draft = rng.integers(0, cfg.vocab, B).astype(np.int32), rng.integers(0, cfg.vocab, B).astype(np.int32)
    rows = int(gam.sum()) + B
    q = torch.randn((rows, cfg.n_heads, cfg.head_dim), generator=g).to(torch.bfloat16).cuda()
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()

    def call(lo, hi, what):
        off = np.concatenate([[0], np.cumsum(gam[lo:hi])]).astype(np.int32)
        k, v = kp.clone(), vp.clone()
        d = draft[lo:hi][gam[lo:hi] > 0] if gam[lo:hi].any() else np.zeros(1, np.int32)
        batch = fv.DeviceBatch(t(L[lo:hi]), t(last[lo:hi]), t(off), t(d), None, None, None, None, t(pt[lo:hi]), k, v, n,
                               np.ascontiguousarray(L[lo:hi]), off)
        if what == "attention":
            r0 = int(gam[:lo].sum()) + lo
            return ctx.attention(0, q[r0:r0 + int(off[-1]) + hi - lo].contiguous(), batch), None, None
        return ctx.prefill(batch, want_logits=True), k, v

    first = np.concatenate([[0], np.cumsum(gam + 1)])
    few = [(lo, min(lo + 250, B)) for lo in range(0, B, 250)]
    # attention: one part per short request, the same bits; long ones may be cut into other parts, merged in fp32, stored in fp16
    whole = call(0, B, "attention")[0]
    for lo, hi in few:
        part = call(lo, hi, "attention")[0]
        for b in range(lo, hi):
            a, c = whole[first[b]:first[b + 1]], part[first[b] - first[lo]:first[b + 1] - first[lo]]
            if L[b] < 128:
                assert torch.equal(a, c), b
            else:
                assert (a - c).abs().max() <= 2.0 ** -9 * a.abs().max(), b
    # the forward: positions, tokens and pages.  Other row counts, other summation orders, other roundings to 16 bits: the bar of
    # the bf16 path; a row of another request, position or token is off by its own size
    logits, k, v = call(0, B, "prefill")
    merged = [kp.clone(), vp.clone()]
    for lo, hi in few:
        part, k1, v1 = call(lo, hi, "prefill")
        a = logits[first[lo]:first[hi]]
        assert ((a - part).norm(dim=1) <= 2e-2 * a.norm(dim=1)).all(), (lo, hi)
        for m, old, new in ((merged[0], kp, k1), (merged[1], vp, v1)):
            m[new != old] = new[new != old]
    for whole_pool, m in ((k, merged[0]), (v, merged[1])):
        d = (whole_pool.float() - m.float()).abs()
        assert d.max() <= 2e-2 * whole_pool.float().abs().max()
    ctx.close()
