"""GPU parity of the accept / resample step (fsv_sample) against the oracle on identical logits.

Logits are seeded inputs (the rejection-sampling configuration: bf16 logits ~ N(0,3), fp32 draft
laws from noised logits, ragged gamma), so both sides see the same bits.  Bar: accepted lengths and
emitted tokens match exactly, except draws the oracle places within 1e-4 of an acceptance threshold
(or within 1e-6 of a CDF edge), which are counted.
"""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_00644_amd import synth
from tests.helpers import compare_decisions

pytestmark = pytest.mark.gpu


def _ctx(vocab, max_batch, max_gamma):
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, vocab, "bf16")
    return fv, fv.Context(cfg, None, max_batch, max_gamma, sampler_only=True)


def _run(fv, ctx, case, temperature=None):
    B = len(case.draft_offsets) - 1
    temp = case.temperature if temperature is None else np.asarray(temperature, np.float32)
    dev = "cuda"
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=dev)
    batch = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.to(dev),
                           t(case.u_accept), t(case.u_sample), t(temp), None, None, None, 0, None,
                           np.ascontiguousarray(case.draft_offsets), np.ascontiguousarray(temp))
    res = fv.DeviceResult.alloc(B)
    ctx.sample(case.logits.to(dev), batch, res)
    torch.cuda.synchronize()
    return res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy(), res.flags.cpu().numpy()


def _oracle(case, temperature=None):
    B = len(case.draft_offsets) - 1
    out = []
    lg = case.logits.float().numpy().astype(np.float64)
    q = case.draft_probs.numpy()
    for b in range(B):
        o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
        T = float(case.temperature[b] if temperature is None else temperature[b])
        s = oracle.sample(lg[o + b: e + b + 1], case.draft_tokens[o:e], q[o:e], case.u_accept[o:e],
                          float(case.u_sample[b]), T)
        out.append(type("R", (), {"sample": s})())
    return out


@pytest.mark.parametrize("vocab,batch,gmax,sigma,dtype,seed", [
    (4096, 5, 4, 0.5, "bf16", 1),          # exactly two sub-blocks
    (5000, 9, 8, 0.7, "bf16", 2),          # ragged tail, vector loads still aligned
    (5003, 7, 6, 1.0, "f32", 3),           # odd vocabulary: scalar loads
    (30000, 6, 16, 0.3, "f32", 4),         # several chunks, gamma at the maximum
    (152064, 12, 16, 1.5, "bf16", 5),      # the full vocabulary of the sampling configuration
])
def test_sampler_matches_oracle(vocab, batch, gmax, sigma, dtype, seed):
    fv, ctx = _ctx(vocab, batch, 16)
    case = synth.make_sampler_case(batch, 1, gmax, vocab, sigma, 0.7, seed, logits_dtype=dtype)
    tau, nxt, flags = _run(fv, ctx, case)
    exp = _oracle(case)
    bad, excused, flagged = compare_decisions(exp, tau, nxt)
    print(f"V={vocab} B={batch}: acceptance {tau.sum()}/{case.draft_offsets[-1]}, flagged {flagged}, excused {excused}")
    assert not bad, bad
    # the library's own residual flag agrees with the oracle wherever the decision matched
    for b, e in enumerate(exp):
        if int(tau[b]) == e.sample.tau and e.sample.accept_margin > 1e-4:
            assert bool(flags[b] & 4) == e.sample.used_residual
    ctx.close()


def test_greedy_and_mixed_temperatures():
    vocab, batch = 9000, 10
    fv, ctx = _ctx(vocab, batch, 16)
    case = synth.make_sampler_case(batch, 0, 6, vocab, 0.2, 1.0, 11, logits_dtype="bf16")
    # bf16 logits over 9000 ids do tie: the lowest id must win on both sides
    temp = np.array([0.0, 1.0] * 5, np.float32)
    # make drafts of greedy requests follow the argmax for a while
    lg = case.logits.float().numpy()
    for b in range(0, batch, 2):
        o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
        for i in range(e - o):
            if i < 2:
                case.draft_tokens[o + i] = int(lg[o + b + i].argmax())
    tau, nxt, flags = _run(fv, ctx, case, temp)
    exp = _oracle(case, temp)
    bad, excused, flagged = compare_decisions(exp, tau, nxt)
    assert not bad, bad
    for b in range(0, batch, 2):
        assert int(tau[b]) == exp[b].sample.tau and int(nxt[b]) == exp[b].sample.next_token   # integer work: exact
        assert flags[b] == 0
    ctx.close()


def test_all_accepted_when_p_equals_q_and_zero_residual_falls_back_to_p():
    vocab, batch, gamma = 4096, 4, 5
    fv, ctx = _ctx(vocab, batch, 16)
    off = np.arange(batch + 1, dtype=np.int32) * gamma
    G, M = batch * gamma, batch * (gamma + 1)
    logits = torch.zeros((M, vocab), dtype=torch.float32)           # p = 1/4096 exactly
    q = torch.full((G, vocab), 1.0 / vocab, dtype=torch.float32)
    q[gamma:2 * gamma] *= 1.0 + 2.0 ** -10                           # request 1: q a hair above p everywhere
    rng = np.random.default_rng(0)
    u = (rng.integers(0, 1 << 24, G) / float(1 << 24)).astype(np.float32)
    u[:gamma] = 1.0 - 2.0 ** -24
    u[gamma] = 1.0 - 2.0 ** -24                                      # request 1 rejects its first draft
    case = synth.SamplerCase(logits, q, rng.integers(0, vocab, G).astype(np.int32), off, u,
                             np.array([0.5, 0.25, 0.0, 0.999], np.float32), np.ones(batch, np.float32))
    tau, nxt, flags = _run(fv, ctx, case)
    exp = _oracle(case)
    assert list(tau) == [gamma, 0, gamma, gamma]
    assert [e.sample.tau for e in exp] == list(tau)
    assert [e.sample.next_token for e in exp] == list(nxt)
    assert nxt[0] == 2048 and nxt[1] == 1024 and nxt[2] == 0
    assert not (flags[1] & 4) and not exp[1].sample.used_residual    # no residual mass: drawn from p
    ctx.close()


def test_empty_batch_and_capacity_errors():
    fv, ctx = _ctx(4096, 4, 8)
    case = synth.make_sampler_case(4, 1, 4, 4096, 0.5, 0.7, 21)
    # gamma beyond the context's capacity is refused on the host, nothing is launched
    big = synth.make_sampler_case(4, 9, 9, 4096, 0.5, 0.7, 22)
    with pytest.raises(fv.FsvError) as ei:
        _run(fv, ctx, big)
    assert ei.value.status == -2
    big5 = synth.make_sampler_case(5, 1, 2, 4096, 0.5, 0.7, 23)
    with pytest.raises(fv.FsvError) as ei:
        _run(fv, ctx, big5)
    assert ei.value.status == -2
    # an empty batch is a no-op
    empty = synth.SamplerCase(case.logits[:0], case.draft_probs[:0], np.zeros(0, np.int32), np.zeros(1, np.int32),
                              np.zeros(0, np.float32), np.zeros(0, np.float32), np.zeros(0, np.float32))
    B0 = fv.DeviceBatch(None, None, torch.zeros(1, dtype=torch.int32, device="cuda"), None, None, None, None, None,
                        None, None, None, 0, None, np.zeros(1, np.int32), None)
    ctx.sample(torch.zeros((1, 4096), device="cuda"), B0, fv.DeviceResult.alloc(1))
    ctx.close()


@pytest.mark.parametrize("vocab,batch,gmax,dtype,seed,scale", [
    (5000, 8, 6, "bf16", 21, 1.0),        # bf16 logits: many tokens tie at the cut value
    (5003, 6, 5, "f32", 22, 1.0),         # odd vocabulary, fp32 keys (three digits)
    (30000, 6, 8, "f32", 23, 1.0),
    (152064, 10, 12, "bf16", 24, 1.0),    # the full vocabulary of the sampling configuration
    (5000, 9, 6, "bf16", 25, 0.02),       # nearly flat laws: the cut lies among the negative logits, far below the
    (40000, 6, 8, "bf16", 26, 0.05),      # window of the one-pass kernel, so these rows take the full passes
])
def test_nucleus_cut_matches_oracle(vocab, batch, gmax, dtype, seed, scale):
    """top-p per request (Regime B samples with top-p): 1.0 (off), 0.9 and a tight 0.5 mixed in one batch."""
    fv, ctx = _ctx(vocab, batch, 16)
    case = synth.make_sampler_case(batch, 1, gmax, vocab, 0.5, 0.7, seed, logits_dtype=dtype)
    if scale != 1.0:
        case.logits = (case.logits.float() * scale).to(case.logits.dtype)
    top_p = np.array([(1.0, 0.9, 0.5)[b % 3] for b in range(batch)], np.float32)
    B = batch
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    bt = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.cuda(),
                        t(case.u_accept), t(case.u_sample), t(case.temperature), None, None, None, 0, None,
                        np.ascontiguousarray(case.draft_offsets), np.ascontiguousarray(case.temperature),
                        t(top_p), top_p)
    res = fv.DeviceResult.alloc(B)
    ctx.sample(case.logits.cuda(), bt, res)
    torch.cuda.synchronize()
    tau, nxt, flags = res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy(), res.flags.cpu().numpy()
    lg = case.logits.float().numpy().astype(np.float64)
    q = case.draft_probs.numpy()
    exp, near = [], 0
    for b in range(B):
        o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
        s = oracle.sample(lg[o + b: e + b + 1], case.draft_tokens[o:e], q[o:e], case.u_accept[o:e],
                          float(case.u_sample[b]), 0.7, top_p=float(top_p[b]))
        if s.nucleus_margin < 1e-6:       # the cut itself is within rounding of top_p: either neighbour is right
            near += 1
            exp.append(None)
        else:
            exp.append(type("R", (), {"sample": s})())
    bad, excused, flagged = compare_decisions(exp, tau, nxt)
    changed = 0
    for b in range(B):    # the cut must matter for some request, or the test shows nothing
        o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
        s0 = oracle.sample(lg[o + b: e + b + 1], case.draft_tokens[o:e], q[o:e], case.u_accept[o:e],
                           float(case.u_sample[b]), 0.7)
        if exp[b] is not None and (s0.tau, s0.next_token) != (exp[b].sample.tau, exp[b].sample.next_token):
            changed += 1
    print(f"V={vocab}: accepted {tau.sum()}/{case.draft_offsets[-1]}, requests the cut changes {changed}, "
          f"near the cut {near}, flagged {flagged}, excused {excused}")
    assert not bad, bad
    assert changed >= 1
    for b in range(B):
        if top_p[b] == 1.0:
            assert not (flags[b] & 8)
    ctx.close()


def test_nucleus_rejects_bad_top_p():
    fv, ctx = _ctx(4096, 2, 4)
    case = synth.make_sampler_case(2, 1, 3, 4096, 0.5, 0.7, 3, logits_dtype="bf16")
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    for bad in (np.array([0.9, 0.0], np.float32), np.array([1.5, 0.9], np.float32)):
        bt = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.cuda(),
                            t(case.u_accept), t(case.u_sample), t(case.temperature), None, None, None, 0, None,
                            np.ascontiguousarray(case.draft_offsets), np.ascontiguousarray(case.temperature), t(bad), bad)
        with pytest.raises(fv.FsvError) as ei:
            ctx.sample(case.logits.cuda(), bt, fv.DeviceResult.alloc(2))
        assert ei.value.status == -1
    ctx.close()


def test_many_small_seeded_cases_against_oracle():
    """Eighty small seeded cases sweeping vocabulary size (aligned and ragged), logit type, gamma, temperature,
    draft noise and top-p, mixed greedy / sampling requests: decisions equal the oracle's except flagged draws."""
    fv = None
    rng = np.random.default_rng(2024)
    total = flagged_total = excused_total = 0
    ctxs = {}
    for case_no in range(80):
        vocab = int(rng.choice([257, 1000, 2048, 2056, 4099, 8192, 8200, 12345]))
        batch = int(rng.integers(1, 9))
        gmax = int(rng.integers(0, 17))
        dtype = "bf16" if rng.random() < 0.5 else "f32"
        sigma = float(rng.choice([0.0, 0.3, 0.8, 1.5]))
        T = float(rng.choice([0.5, 0.7, 1.0, 1.3]))
        if vocab not in ctxs:
            fv, ctxs[vocab] = _ctx(vocab, 8, 16)
        ctx = ctxs[vocab]
        case = synth.make_sampler_case(batch, 0, gmax, vocab, sigma, T, 1000 + case_no, logits_dtype=dtype)
        temp = np.where(rng.random(batch) < 0.2, 0.0, T).astype(np.float32)        # some greedy requests
        top_p = rng.choice([1.0, 1.0, 0.95, 0.8, 0.4], size=batch).astype(np.float32)
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
        bt = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.cuda(),
                            t(case.u_accept), t(case.u_sample), t(temp), None, None, None, 0, None,
                            np.ascontiguousarray(case.draft_offsets), temp, t(top_p), top_p)
        res = fv.DeviceResult.alloc(batch)
        ctx.sample(case.logits.cuda(), bt, res)
        torch.cuda.synchronize()
        tau, nxt = res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy()
        lg = case.logits.float().numpy().astype(np.float64)
        q = case.draft_probs.numpy()
        exp = []
        for b in range(batch):
            o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
            s = oracle.sample(lg[o + b: e + b + 1], case.draft_tokens[o:e], q[o:e], case.u_accept[o:e],
                              float(case.u_sample[b]), float(temp[b]), top_p=float(top_p[b]))
            exp.append(None if s.nucleus_margin < 1e-6 else type("R", (), {"sample": s})())
        bad, excused, flagged = compare_decisions(exp, tau, nxt)
        assert not bad, (case_no, vocab, batch, dtype, T, bad)
        total += batch
        flagged_total += flagged
        excused_total += excused
    print(f"{total} requests in 80 cases: flagged {flagged_total}, excused {excused_total}")
    for c in ctxs.values():
        c.close()


@pytest.mark.parametrize("vocab,batch,gmax,dtype,seed", [
    (5000, 9, 6, "bf16", 41),        # bf16 logits: the k-th value is usually shared by several tokens (ties kept)
    (5003, 8, 5, "f32", 42),         # odd vocabulary, fp32 keys (three digits)
    (152064, 12, 12, "bf16", 43),    # the full vocabulary of the sampling configuration
    (5000, 16, 6, "bf16", 44),       # more requests: every entry of the list below occurs, the deep cuts twice
])
def test_top_k_cut_matches_oracle(vocab, batch, gmax, dtype, seed):
    """top-k per request, alone and followed by top-p, mixed with uncut and greedy requests in one batch.  The k-th
    token of the large k lies among the negative logits: below the window of the one-pass kernel for bf16 logits, so
    those rows take the full passes."""
    fv, ctx = _ctx(vocab, batch, 16)
    case = synth.make_sampler_case(batch, 1, gmax, vocab, 0.5, 0.7, seed, logits_dtype=dtype)
    top_k = np.array([(0, 50, 5, 1, 2000, vocab + 7, (vocab * 4) // 5, (vocab * 9) // 10)[b % 8] for b in range(batch)], np.int32)
    top_p = np.array([(1.0, 1.0, 0.8, 1.0, 0.9, 0.9, 1.0, 0.999)[b % 8] for b in range(batch)], np.float32)
    temp = case.temperature.copy()
    if batch > 7:
        temp[7] = 0.0                 # a greedy request ignores both cuts
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    bt = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.cuda(),
                        t(case.u_accept), t(case.u_sample), t(temp), None, None, None, 0, None,
                        np.ascontiguousarray(case.draft_offsets), np.ascontiguousarray(temp),
                        t(top_p), top_p, t(top_k), top_k)
    res = fv.DeviceResult.alloc(batch)
    ctx.sample(case.logits.cuda(), bt, res)
    torch.cuda.synchronize()
    tau, nxt = res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy()
    lg = case.logits.float().numpy().astype(np.float64)
    q = case.draft_probs.numpy()
    exp, near, changed = [], 0, 0
    for b in range(batch):
        o, e = int(case.draft_offsets[b]), int(case.draft_offsets[b + 1])
        args = (lg[o + b: e + b + 1], case.draft_tokens[o:e], q[o:e], case.u_accept[o:e], float(case.u_sample[b]), float(temp[b]))
        s = oracle.sample(*args, top_p=float(top_p[b]), top_k=int(top_k[b]))
        if s.nucleus_margin < 1e-6:
            near += 1
            exp.append(None)
            continue
        exp.append(type("R", (), {"sample": s})())
        s0 = oracle.sample(*args)
        changed += (s0.tau, s0.next_token) != (s.tau, s.next_token)
    bad, excused, flagged = compare_decisions(exp, tau, nxt)
    print(f"V={vocab}: accepted {tau.sum()}/{case.draft_offsets[-1]}, requests the cut changes {changed}, near {near}, "
          f"flagged {flagged}, excused {excused}")
    assert not bad, bad
    assert changed >= 1
    # the static entry point takes the same fields
    res2 = fv.DeviceResult.alloc(batch)
    fv.sample_static(vocab, case.logits.cuda(), bt, res2)
    torch.cuda.synchronize()
    assert torch.equal(res2.accepted_len, res.accepted_len) and torch.equal(res2.next_token, res.next_token)
    ctx.close()


def test_windowed_and_full_nucleus_passes_agree(monkeypatch):
    """The one-pass windowed cut (bf16 logits) and the digit-by-digit passes are two routes to the same cut: on the
    full-vocabulary case, with top-p and top-k mixed, they must give the same decisions and flags, except where a
    cut is flagged as within rounding of top_p (the windowed pass measures top_p against the statistics pass's
    normaliser, the full passes against their own integer sum)."""
    V, B = 152064, 24
    fv, ctx = _ctx(V, B, 16)
    case = synth.make_sampler_case(B, 1, 12, V, 0.7, 0.7, 77, logits_dtype="bf16")
    top_p = np.array([(0.9, 0.5, 1.0, 0.99, 0.95, 0.9)[b % 6] for b in range(B)], np.float32)
    top_k = np.array([(0, 0, 40, 0, 1000, 7)[b % 6] for b in range(B)], np.int32)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    bt = fv.DeviceBatch(None, None, t(case.draft_offsets), t(case.draft_tokens), case.draft_probs.cuda(),
                        t(case.u_accept), t(case.u_sample), t(case.temperature), None, None, None, 0, None,
                        np.ascontiguousarray(case.draft_offsets), np.ascontiguousarray(case.temperature),
                        t(top_p), top_p, t(top_k), top_k)
    lg = case.logits.cuda()
    out = {}
    for mode in ("0", "1"):
        monkeypatch.setenv("FSV_NUCLEUS_FULL", mode)
        res = fv.DeviceResult.alloc(B)
        ctx.sample(lg, bt, res)
        torch.cuda.synchronize()
        out[mode] = (res.accepted_len.cpu().numpy(), res.next_token.cpu().numpy(), res.flags.cpu().numpy())
    near = (out["0"][2] | out["1"][2]) & 8
    same = (out["0"][0] == out["1"][0]) & (out["0"][1] == out["1"][1])
    print(f"requests whose cut is flagged near: {int((near != 0).sum())} of {B}; identical decisions: {int(same.sum())}")
    assert bool((same | (near != 0)).all())
    assert int((near != 0).sum()) <= B // 4
    ctx.close()


# Residual masses 2^-17 - q of one id in each of the first twelve 2048-id sub-blocks, for which half the total lies between two
# roundings of the same running mass: the mass of the first six sub-blocks added one after the other, and as lane sums and
# their scan (the two ways the selection meets it).
_GAPS = [
    "0x1.13e4bep-44 0x1.6a26e2p-44 0x1.482808p-47 0x1.bc071cp-44 0x1.bfd1bcp-45 0x1.b60d74p-55 0x1.eca9fap-54 0x1.ee9b76p-45 "
    "0x1.2f4528p-55 0x1.1d6c38p-44 0x1.21e25cp-46 0x1.72b1e2p-43",
    "0x1.d63cfep-48 0x1.3b78c2p-49 0x1.95acfap-46 0x1.bfae74p-50 0x1.6a15bap-45 0x1.a4c9d4p-55 0x1.1e52b6p-52 0x1.b9cb40p-53 "
    "0x1.4dc476p-51 0x1.1532f0p-44 0x1.4b9ee6p-54 0x1.76637ap-47",
    "0x1.188aa2p-55 0x1.873d84p-47 0x1.fc9fa8p-52 0x1.39fbeep-46 0x1.44d676p-46 0x1.c70d20p-54 0x1.3043d2p-52 0x1.2b8a42p-48 "
    "0x1.37370cp-53 0x1.93c33ep-51 0x1.80f2b0p-51 0x1.70ffa6p-45",
]


@pytest.mark.parametrize("place", [0, 9, 1000, 2047])
def test_emitted_id_has_mass_when_the_target_falls_between_two_roundings(place):
    V, B = 1 << 17, len(_GAPS)
    fv, ctx = _ctx(V, B, 16)
    p = 2.0 ** -17                                   # equal logits: every probability is exactly this
    q = torch.full((B, V), p, dtype=torch.float32)   # no residual
    for b, law in enumerate(_GAPS):
        for sb, x in enumerate(law.split()):
            q[b, sb * 2048 + place] = float.fromhex(x)
    d = V - 1                                        # the draft, rejected: p / q = 1/2 < u
    q[:, d] = 2.0 * p
    off = np.arange(B + 1, dtype=np.int32)
    case = synth.SamplerCase(torch.zeros((2 * B, V)), q, np.full(B, d, np.int32), off, np.full(B, 0.75, np.float32),
                             np.full(B, 0.5, np.float32), np.ones(B, np.float32))
    tau, nxt, flags = _run(fv, ctx, case)
    assert list(tau) == [0] * B
    for b in range(B):
        assert float(q[b, int(nxt[b])]) < p, (b, int(nxt[b]))      # an id of zero residual was emitted
        assert int(nxt[b]) in (5 * 2048 + place, 6 * 2048 + place)  # either side of the edge the target sits on
        assert (int(flags[b]) & 6) == 6                             # residual draw, flagged as close to an edge
    ctx.close()
