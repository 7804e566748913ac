"""The law kernel of fsv_draft_probs at the edges of its blocks (4096 ids), of the statistics' chunks (8192 ids) and of its
16-byte loads, against softmax(z / T) in fp64 of the logits the same call returns."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [256, 4093, 4096, 4100, 8192, 8193, 16388, 24571])
@pytest.mark.parametrize("greedy", [False, True])
def test_law_is_the_softmax_of_the_logits(vocab, greedy):
    from paper_2601_00644_amd import flexverify as fv
    cfg = dataclasses.replace(synth.MODELS["mini64"], vocab=vocab)
    w = synth.make_weights(cfg, 3, std=0.05)
    gam, L = np.array([0, 3, 7, 1], np.int32), np.array([4, 0, 33, 18], np.int32)
    off = np.concatenate([[0], np.cumsum(gam)]).astype(np.int32)
    B, G = 4, int(off[-1])
    pt, n = synth.make_page_table(L, gam, 16, "interleaved", 1)
    ctx = fv.Context(cfg, {k: t.cuda() for k, t in w.items()}, max_batch=B, max_gamma=8, max_pages_per_req=pt.shape[1])
    ctx.draft_attach({k: t.cuda() for k, t in synth.make_draft_head(cfg, 256, 256, 4, std=0.2).items()})
    kp, vp = fv.alloc_draft_pools(cfg, n)
    T = np.array([0.7, 1.0, 0.0 if greedy else 0.5, 1.3], np.float32)
    t = lambda a: torch.as_tensor(a).cuda()
    rng = np.random.default_rng(2)
    batch = fv.DeviceBatch(t(L), t(rng.integers(0, vocab, B).astype(np.int32)), t(off), t(rng.integers(0, vocab, G).astype(np.int32)),
                           None, None, None, t(T), t(pt), kp, vp, n, L, off, T)
    for mode, rows in ((fv.DRAFT_Q_VERIFY, [(int(off[b]) + i, int(off[b]) + b + i, b) for b in range(B) for i in range(gam[b])]),
                       (fv.DRAFT_Q_ALL, [(int(off[b]) + b + i, int(off[b]) + b + i, b) for b in range(B) for i in range(gam[b] + 1)])):
        q, z = ctx.draft_probs(batch, mode, want_logits=True)
        q, z = q.double().cpu(), z.double().cpu()
        for qi, r, b in rows:
            if T[b] == 0:
                assert not q[qi].any()            # left untouched: zeros
                continue
            want = torch.softmax(z[r] / float(T[b]), -1)
            # exponent (z - max) / T rounded to fp32: a relative 2^-23 of up to |z - max| / T, twice (argument, 2^x), and the sum
            bound = (4 + (z[r].max() - z[r]) / float(T[b])) * 2.0 ** -22
            assert ((q[qi] - want).abs() <= want * bound + 1e-30).all()
    ctx.close()


@pytest.mark.parametrize("vocab,at", [(8193, 8192), (8200, 8195), (16384, 100), (16388, 16387)])
def test_a_nan_logit_makes_the_law_nan(vocab, at):
    """As softmax does, also where the NaN is alone in its chunk of 8192 ids (8193: the last id has one to itself)."""
    from paper_2601_00644_amd import flexverify as fv
    cfg = dataclasses.replace(synth.MODELS["mini64"], vocab=vocab)
    w = synth.make_weights(cfg, 3, std=0.05)
    gam, L = np.array([2, 1], np.int32), np.array([4, 18], np.int32)
    off = np.array([0, 2, 3], np.int32)
    pt, n = synth.make_page_table(L, gam, 16, "interleaved", 1)
    ctx = fv.Context(cfg, {k: t.cuda() for k, t in w.items()}, max_batch=2, max_gamma=8, max_pages_per_req=pt.shape[1])
    head = synth.make_draft_head(cfg, 256, 256, 4, std=0.2)
    head["wv"][at] = float("nan")
    ctx.draft_attach({k: t.cuda() for k, t in head.items()})
    kp, vp = fv.alloc_draft_pools(cfg, n)
    T = np.array([0.7, 1.0], np.float32)
    t = lambda a: torch.as_tensor(a).cuda()
    batch = fv.DeviceBatch(t(L), t(np.array([1, 2], np.int32)), t(off), t(np.array([5, 6, 7], np.int32)), None, None, None, t(T), t(pt), kp,
                           vp, n, L, off, T)
    for mode in (fv.DRAFT_Q_VERIFY, fv.DRAFT_Q_ALL):
        q, z = ctx.draft_probs(batch, mode, want_logits=True)
        assert z[:, at].isnan().all() and int(z.isnan().sum()) == z.shape[0]
        assert q.isnan().all()
    ctx.close()
