"""The fp32 path's kernels off their usual sizes: row counts around the blocks of eight, contraction lengths that do not take
16-byte loads, unaligned inputs, head sizes around the blocks of 512 threads, key counts around the pages.  Single kernels
against fp64, the whole forward (normalised and SwiGLU projections) against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


def _ctx(cfg, w, **kw):
    from paper_2601_00644_amd import flexverify as fv
    return fv, fv.Context(cfg, {k: v.cuda() for k, v in w.items()}, **kw)


@pytest.mark.parametrize("M", [1, 7, 8, 9, 40])
@pytest.mark.parametrize("d,F,shift", [(64, 96, 0), (70, 33, 0), (64, 96, 1), (130, 1027, 0)])
def test_linear(M, d, F, shift):
    cfg = synth.ModelCfg("f32odd", 2, d, 2, 1, 34, F, 131, "f32")
    w = synth.make_weights(cfg, M, std=0.3)
    fv, ctx = _ctx(cfg, w, max_batch=4, max_gamma=9, max_pages_per_req=4, max_rows=40)
    g = torch.Generator().manual_seed(M)
    for wh, key, K in [(fv.W_QKV, "w_qkv.1", d), (fv.W_O, "w_o.0", 68), (fv.W_GATE_UP, "w_gate_up.1", d), (fv.W_DOWN, "w_down.0", F),
                       (fv.W_LM_HEAD, "lm_head", d)]:
        x = torch.randn((M, K), generator=g)
        buf = torch.zeros(M * K + 4).cuda()
        xs = buf[shift:shift + M * K].view(M, K)
        xs.copy_(x)
        y = ctx.linear(wh, int(key.split(".")[1]) if "." in key else 0, xs, w[key].shape[0]).double().cpu()
        ref = x.double() @ w[key].double().t()
        bound = (x.double().abs() @ w[key].double().abs().t()) * (K / 64 + 16) * 2.0 ** -24   # a lane's chain, then ten adds
        assert ((y - ref).abs() <= bound).all(), (key, M)
    ctx.close()


@pytest.mark.parametrize("hd,heads,kv", [(2, 4, 2), (34, 3, 1), (64, 4, 4), (254, 2, 1), (256, 2, 2), (300, 2, 1), (512, 1, 1), (514, 2, 1)])
def test_attention(hd, heads, kv):
    cfg = synth.ModelCfg("f32att", 1, 32, heads, kv, hd, 32, 64, "f32")
    L, gam = np.array([0, 15, 16, 130, 700], np.int32), np.array([0, 1, 3, 2, 4], np.int32)
    off = np.concatenate([[0], np.cumsum(gam)]).astype(np.int32)
    pt, n = synth.make_page_table(L, gam, 16, "permuted", 1)
    fv, ctx = _ctx(cfg, synth.make_weights(cfg, 1), max_batch=5, max_gamma=4, max_pages_per_req=pt.shape[1])
    kp, vp = fv.alloc_pools(cfg, n)
    t = lambda a: torch.as_tensor(a).cuda()
    g = torch.Generator().manual_seed(hd)
    q = torch.randn((int(off[-1]) + 5, heads, hd), generator=g)
    ks = [torch.randn((1, int(L[b] + gam[b]) + 1, kv, hd), generator=g) for b in range(5)]
    vs = [torch.randn_like(k) for k in ks]
    for b in range(5):
        ctx.kv_import(kp, vp, n, t(pt)[b], 0, ks[b].cuda(), vs[b].cuda())
    batch = fv.DeviceBatch(t(L), None, t(off), None, None, None, None, None, t(pt), kp, vp, n, L, off)
    out = ctx.attention(0, q.cuda(), batch).double().cpu().view(-1, heads, hd)
    for b in range(5):
        for i in range(int(gam[b]) + 1):
            r, nk = int(off[b]) + b + i, int(L[b]) + i + 1
            for h in range(heads):
                k, v = ks[b][0, :nk, h * kv // heads].double(), vs[b][0, :nk, h * kv // heads].double()
                p = torch.softmax((k @ q[r, h].double()) / hd ** 0.5, -1)
                # scores of size |s| rounded to 2^-24 move a probability by that much; values of unit size, sums of nk terms
                bound = (4 + (k @ q[r, h].double()).abs().max() / hd ** 0.5 + hd / 16 + nk / 64) * 2.0 ** -22
                assert (out[r, h] - p @ v).abs().max() <= bound * max(1.0, float(v.abs().max())), (b, i, h)
    ctx.close()


@pytest.mark.parametrize("rows", [1, 8, 21])
def test_forward_of_odd_sizes(rows):
    cfg = synth.ModelCfg("f32odd", 2, 70, 3, 1, 34, 46, 131, "f32")
    w = synth.make_weights(cfg, 9, std=0.2)
    fv, ctx = _ctx(cfg, w, max_batch=4, max_gamma=8, max_pages_per_req=4)
    toks = np.random.default_rng(rows).integers(0, cfg.vocab, rows).astype(np.int32)
    kp, vp = fv.alloc_pools(cfg, 4)
    got = ctx.prefill(fv.prefill_pieces([(0, 0, toks)], np.array([[2, 0, 3, 1]], np.int32), kp, vp, 4, 9), want_logits=True).cpu().numpy()
    k, v = oracle.new_cache(cfg, rows)
    ref = oracle.forward(cfg, synth.weights_to_numpy(cfg, w), k, v, 0, toks)
    rms = np.sqrt((ref ** 2).mean(1, keepdims=True))
    assert (np.abs(got - ref) <= 1e-4 * np.maximum(np.abs(ref), rms)).all()      # the fp32 path's bar
    ctx.close()


def test_one_row_alone_gives_the_bits_it_gives_in_a_batch():
    """A call of one row takes its own form of the projections: same sums, same order."""
    cfg = synth.MODELS["minif32"]
    w = synth.make_weights(cfg, 5, std=0.1)
    fv, ctx = _ctx(cfg, w, max_batch=9, max_gamma=0, max_pages_per_req=2)
    toks = np.random.default_rng(1).integers(0, cfg.vocab, 9).astype(np.int32)
    pt = np.arange(18, dtype=np.int32).reshape(9, 2)
    t = lambda a: torch.as_tensor(a).cuda()

    def prefill(rows):
        kp, vp = fv.alloc_pools(cfg, 18)
        n = len(rows)
        L, off = np.zeros(n, np.int32), np.zeros(n + 1, np.int32)
        return ctx.prefill(fv.DeviceBatch(t(L), t(toks[rows]), t(off), None, None, None, None, None, t(pt[rows]), kp, vp, 18, L, off),
                           want_logits=True).cpu()

    together = prefill(np.arange(9))
    for r in (0, 4, 8):
        assert torch.equal(prefill(np.array([r]))[0], together[r])
    ctx.close()


@pytest.mark.parametrize("hd,heads,kv", [(2, 16, 2), (34, 12, 3), (64, 16, 4), (128, 8, 2)])
def test_attention_of_many_blocks_with_few_keys(hd, heads, kv):
    """2048 blocks or more of up to 64 keys take smaller blocks: the bits of the same rows in a call that takes the larger ones,
    and (one request of each length) the fp64 result."""
    cfg = synth.ModelCfg("f32few", 1, 32, heads, kv, hd, 32, 64, "f32")
    B = 2048 // heads
    L = np.array([0, 1, 14, 15, 16, 31, 62, 63], np.int32)[np.arange(B) % 8]
    gam, off = np.zeros(B, np.int32), np.zeros(B + 1, np.int32)
    pt, n = synth.make_page_table(L, gam, 16, "permuted", 1)
    fv, ctx = _ctx(cfg, synth.make_weights(cfg, 1), max_batch=B, max_gamma=0, max_pages_per_req=pt.shape[1])
    kp, vp = fv.alloc_pools(cfg, n)
    g = torch.Generator().manual_seed(hd)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    q = torch.randn((B, heads, hd), generator=g)
    kv_of = {b: [torch.randn((1, int(L[b]) + 1, kv, hd), generator=g) for _ in range(2)] for b in range(B)}
    for b, (k, v) in kv_of.items():
        ctx.kv_import(kp, vp, n, t(pt)[b], 0, k.cuda(), v.cuda())

    def run(rows):
        o = np.zeros(len(rows) + 1, np.int32)
        return ctx.attention(0, q[rows].cuda(), fv.DeviceBatch(t(L[rows]), None, t(o), None, None, None, None, None, t(pt[rows]), kp, vp, n,
                                                               np.ascontiguousarray(L[rows]), o)).cpu().view(-1, heads, hd)

    out = run(np.arange(B))                     # B * heads = 2048 blocks
    assert torch.equal(run(np.arange(B - 1)), out[:B - 1])     # fewer: the larger blocks
    for b in range(8):
        k, v = (x[0].double() for x in kv_of[b])
        for h in range(heads):
            s = (k[:, h * kv // heads] @ q[b, h].double()) / hd ** 0.5
            ref = torch.softmax(s, -1) @ v[:, h * kv // heads]
            bound = (4 + s.abs().max() + hd / 16 + len(s) / 64) * 2.0 ** -22
            assert (out[b, h].double() - ref).abs().max() <= bound * max(1.0, float(v.abs().max())), (b, h)
    ctx.close()
