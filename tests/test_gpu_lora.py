"""GPU parity of the verification step for an EVOLVED target: per-request LoRA adapters (Sec. IV-A) in one ragged batch.

Requests of one batch use different target versions (adapter 0, 1, 2 ... or the base target); the oracle scores each
request with ITS adapter.  Bar: the bf16 logit bar of helpers.check_bf16_logits (flat 2e-2 against the fp64 oracle),
the layer-0 cache rows bit for bit against the bf16-storage oracle (they carry the adapted q|k|v projection), decisions
exact on identical logits.  The adapters must matter: adapted logits differ from the base target's by far more than
the bar, and a base-target request in the same batch still matches the base oracle.
"""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_00644_amd import synth
from tests.helpers import (STORED_BF16, build_case, check_bf16_kv, check_bf16_logits, compare_decisions, fmt_bf16_report,
                           logit_metrics, oracle_cache_from_context)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,batch,ctx_hi,gmax,rank,seed", [
    ("mini64", 7, 400, 8, 16, 51),      # three layers: two adapted, the last one frozen
    ("mini128", 6, 700, 16, 8, 52),     # two layers, attention output wider than the model (qd = 1024, d = 512)
    ("mini64", 9, 60, 3, 64, 53),       # the largest rank
])
def test_mixed_adapters_in_one_ragged_batch(name, batch, ctx_hi, gmax, rank, seed):
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS[name]
    wl = synth.Workload("t", name, batch, 1, ctx_hi, "uniform", 0, gmax, "uniform", 0.7, 0.8, "permuted")
    case = build_case(cfg, wl, seed=seed, weight_std=0.04, run_oracle=False)
    req = case.req
    n_ad = 3
    adapters = [synth.make_lora(cfg, rank, seed, a) for a in range(n_ad)]
    adapters_np = [synth.lora_to_numpy(cfg, a) for a in adapters]
    ids = np.array([(0, 1, -1, 2, 1, 7)[b % 6] for b in range(batch)], np.int32)     # 7 is out of range: base target
    dev = "cuda"
    ctx = fv.Context(cfg, {k: v.to(dev) for k, v in case.weights.items()}, max_batch=batch, max_gamma=16,
                     max_pages_per_req=req.page_table.shape[1])
    ctx.lora_load([{k: ([t.to(dev) for t in v] if isinstance(v, list) else v) for k, v in a.items()} for a in adapters])
    kp, vp = fv.alloc_pools(cfg, req.num_pages, dev)
    pt = torch.as_tensor(req.page_table, device=dev)
    for b in range(batch):
        if case.ctx_k[b].shape[1] > 0:
            ctx.kv_import(kp, vp, req.num_pages, pt[b], 0, case.ctx_k[b].to(dev), case.ctx_v[b].to(dev))
    bt = fv.device_batch(req, case.draft_tokens, case.draft_probs.to(dev), kp, vp, dev)
    bt.adapter = torch.as_tensor(ids, device=dev)
    res = fv.DeviceResult.alloc(batch, bt.rows, cfg.vocab, want_logits=True)
    ctx.verify(bt, res)
    torch.cuda.synchronize()
    lg = res.logits_out.cpu().numpy().astype(np.float64)
    tau, nxt, nl = res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy(), res.new_seq_lens.cpu().numpy()
    changed = 0
    for b in range(batch):
        L, g, o = int(req.seq_lens[b]), int(req.gammas[b]), int(req.draft_offsets[b])
        lo = adapters_np[ids[b]] if 0 <= ids[b] < n_ad else None
        args = (L, int(req.last_token[b]), case.draft_tokens[o:o + g], case.draft_probs[o:o + g].numpy(),
                req.u_accept[o:o + g], float(req.u_sample[b]), float(req.temperature[b]))
        kc, vc = oracle_cache_from_context(cfg, case.ctx_k[b], case.ctx_v[b], L + g + 1)
        e = oracle.verify(cfg, case.weights_np, kc, vc, *args, lora=lo)
        ks, vs = oracle_cache_from_context(cfg, case.ctx_k[b], case.ctx_v[b], L + g + 1)
        es = oracle.verify(cfg, case.weights_np, ks, vs, *args, stored=STORED_BF16, lora=lo)
        got = lg[o + b: o + b + g + 1]
        rep = check_bf16_logits(got, e.logits, es.logits, f"{name} request {b} adapter {ids[b]}")
        # decisions on identical logits: the oracle's sampler on the library's logits
        s = oracle.sample(got, case.draft_tokens[o:o + g], case.draft_probs[o:o + g].numpy(), req.u_accept[o:o + g],
                          float(req.u_sample[b]), float(req.temperature[b]))
        exp = [None] * batch
        exp[b] = type("R", (), {"sample": s})()
        bad, _, _ = compare_decisions(exp, tau, nxt)
        assert not bad, bad
        # appended cache rows of the valid prefix: layer 0 carries the adapted projection and must match bit for bit
        n_new = int(nl[b]) - L
        gk, gv = ctx.kv_export(kp, vp, req.num_pages, pt[b], L, n_new)
        for nm, gotkv, ref in (("k", gk, ks[:, L:L + n_new]), ("v", gv, vs[:, L:L + n_new])):
            check_bf16_kv(gotkv.float().cpu().numpy().astype(np.float64).reshape(cfg.n_layers, n_new, -1),
                          ref.reshape(cfg.n_layers, n_new, -1), True, (b, nm))
        if lo is not None:
            kb, vb = oracle_cache_from_context(cfg, case.ctx_k[b], case.ctx_v[b], L + g + 1)
            base = oracle.verify(cfg, case.weights_np, kb, vb, *args)
            diff = logit_metrics(e.logits, base.logits)["l2"]
            assert diff > 0.1, (b, diff)                 # the adapter changes the target by far more than the bar
            changed += 1
        if b == 0:
            print(f"{name} rank {rank}: request 0: {fmt_bf16_report(rep)}")
    assert changed >= 3
    # without adapter ids the same context serves the base target
    bt.adapter = None
    res2 = fv.DeviceResult.alloc(batch, bt.rows, cfg.vocab, want_logits=True)
    kp2, vp2 = fv.alloc_pools(cfg, req.num_pages, dev)
    for b in range(batch):
        if case.ctx_k[b].shape[1] > 0:
            ctx.kv_import(kp2, vp2, req.num_pages, pt[b], 0, case.ctx_k[b].to(dev), case.ctx_v[b].to(dev))
    bt.k_pool, bt.v_pool = kp2, vp2
    ctx.verify(bt, res2)
    torch.cuda.synchronize()
    b = int(np.nonzero((ids < 0) | (ids >= n_ad))[0][0])
    o, g = int(req.draft_offsets[b]), int(req.gammas[b])
    assert torch.equal(res2.logits_out[o + b: o + b + g + 1], res.logits_out[o + b: o + b + g + 1])   # a base request is untouched by the others' adapters
    ctx.close()


def test_lora_load_refusals():
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS["mini64"]
    w = synth.make_weights(cfg, 3)
    ctx = fv.Context(cfg, {k: v.cuda() for k, v in w.items()}, 2, 4, 8)
    bad_rank = synth.make_lora(cfg, 12, 1, 0, device="cuda")
    with pytest.raises(fv.FsvError) as ei:
        ctx.lora_load([bad_rank])
    assert ei.value.status == -3
    ctx.lora_load([synth.make_lora(cfg, 8, 1, 0, device="cuda")])
    ctx.lora_load(None)            # removing the adapters again is fine
    ctx.close()


def test_a_base_request_of_a_short_call_is_untouched_by_the_others_adapters():
    """Up to 16 rows: the base request's logits and appended rows keep their bits whether or not the call carries adapter ids."""
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS["mini64"]
    wl = synth.Workload("t", "mini64", 3, 20, 90, "uniform", 3, 4, "uniform", 0.7, 0.8, "permuted")
    case = build_case(cfg, wl, seed=54, weight_std=0.04, run_oracle=False)
    req = case.req
    assert int(req.draft_offsets[-1]) + req.batch <= 16
    ctx = fv.Context(cfg, {k: v.cuda() for k, v in case.weights.items()}, max_batch=3, max_gamma=16, max_pages_per_req=req.page_table.shape[1])
    ctx.lora_load([synth.make_lora(cfg, 16, 54, a, device="cuda") for a in range(2)])
    pt = torch.as_tensor(req.page_table, device="cuda")
    got = []
    for ids in ([1, -1, 0], [-1, -1, -1], None):
        kp, vp = fv.alloc_pools(cfg, req.num_pages, "cuda")
        for b in range(3):
            ctx.kv_import(kp, vp, req.num_pages, pt[b], 0, case.ctx_k[b].cuda(), case.ctx_v[b].cuda())
        bt = fv.device_batch(req, case.draft_tokens, case.draft_probs.cuda(), kp, vp, "cuda")
        bt.adapter = None if ids is None else torch.tensor(ids, dtype=torch.int32, device="cuda")
        res = fv.DeviceResult.alloc(3, bt.rows, cfg.vocab, want_logits=True)
        ctx.verify(bt, res)
        o, g, L = int(req.draft_offsets[1]), int(req.gammas[1]), int(req.seq_lens[1])
        got.append((res.logits_out[o + 1:o + 1 + g + 1].clone(), *ctx.kv_export(kp, vp, req.num_pages, pt[1], L, g + 1)))
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
    ctx.close()
