"""The top-k / top-p cut kernel (fsv_sample) where its fast way can go wrong, against the digit-by-digit way forced with
FSV_NUCLEUS_FULL=1: vocabularies around the rounds of its loads, ragged and unaligned rows, cuts of every depth, laws whose
candidates overflow its list, rows with -inf and NaN.  Both ways form the same integer masses; for bf16 logits the fast way
measures top_p against the statistics' normaliser, which can move a cut only where the call flags it (bit 3)."""
import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


def _laws(kind, M, V, g):
    z = torch.randn((M, V), generator=g)
    if kind == "normal":
        return z * 3.0
    if kind == "flat":                       # thousands of candidates in one bin
        return z * 1e-3
    if kind == "ties":                       # a handful of values
        return (z * 2.0).round()
    if kind == "peaked":
        z[:, 7] += 60.0
        return z
    z = z * 2.0                              # "holes": masked tokens, one row with a NaN, one without any finite logit
    z[:, ::3] = -float("inf")
    z[0, 5] = float("nan")
    z[1] = -float("inf")
    return z


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [64, 8191, 32768, 32776, 65540, 100003])
@pytest.mark.parametrize("kind", ["normal", "flat", "ties", "peaked", "holes"])
def test_fast_cut_equals_the_digit_passes(kind, V, dtype, monkeypatch):
    from paper_2601_00644_amd import flexverify as fv
    B, gam = 6, 2
    off = (np.arange(B + 1) * gam).astype(np.int32)
    g = torch.Generator().manual_seed(V)
    M = B * (gam + 1)
    lg = _laws(kind, M, V, g).to(dtype).cuda()
    q = torch.softmax(torch.randn((B * gam, V), generator=g), -1).cuda()
    T = np.array([0.7, 1.0, 1.3, 0.0, 0.5, 1.0], np.float32)
    t = lambda a: torch.as_tensor(a).cuda()
    rng = np.random.default_rng(V)
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    d = rng.integers(0, V, B * gam).astype(np.int32)
    d[::2] = lg.float()[torch.arange(0, M, 3).cuda()].nan_to_num(nan=-9e9).argmax(-1).cpu().numpy()     # first drafts: likely tokens
    batch = fv.DeviceBatch(None, None, t(off), t(d), q, t(synth.uniforms24(B * gam, V, 1)), t(synth.uniforms24(B, V, 2)), t(T), None,
                           None, None, 0, None, off, T)
    for top_p, top_k in (([0.9] * B, None), ([0.999, 0.5, 0.05, 0.9, 1.0, 0.99], None), (None, [1, 50, 3, 7, V - 1, 0]),
                         ([0.9, 1.0, 0.3, 0.9, 0.95, 0.9], [40, 50, 1000, 5, 0, min(V, 30000)])):
        batch.top_p_host = None if top_p is None else np.asarray(top_p, np.float32)
        batch.top_p = None if top_p is None else t(batch.top_p_host)
        batch.top_k_host = None if top_k is None else np.asarray(top_k, np.int32)
        batch.top_k = None if top_k is None else t(batch.top_k_host)
        out = []
        for full in ("0", "1"):
            monkeypatch.setenv("FSV_NUCLEUS_FULL", full)
            res = fv.DeviceResult.alloc(B)
            ctx.sample(lg, batch, res)
            out.append(torch.stack([res.accepted_len, res.next_token, res.flags]).cpu().numpy())
        a, b = out
        near = ((a[2] | b[2]) & 8) != 0
        if dtype == torch.float32:
            assert (a == b).all(), (top_p, top_k)
        else:
            assert ((a == b).all(0) | near).all(), (top_p, top_k)
    ctx.close()


def test_bf16_top_p_is_measured_against_the_exact_mass(monkeypatch):
    """bf16 rows whose cut lies more than two binades below the maximum: top_p steps by its last bit across the kept mass at the
    end of several groups of equal logits.  The cut has to change at the step at which the digit passes, which sum the row's
    mass as integers, change it; a normaliser rounded to fp32 terms is off by such steps."""
    from paper_2601_00644_amd import flexverify as fv
    V, T, steps = 40000, 1.5, 24
    z = (torch.randn(V, generator=torch.Generator().manual_seed(3)) * 3.0).to(torch.bfloat16)
    v = z.float().sort(descending=True).values.numpy()
    e = np.exp((v.astype(np.float64) - float(v[0])) / T)
    c = np.cumsum(e) / e.sum()
    ends = np.flatnonzero(v[1:] != v[:-1])
    ends = ends[(c[ends] > 0.97) & (c[ends] < 0.995)][::3][:8]
    assert len(ends) == 8 and v[ends[0]] < v[0] / 4          # below the second binade
    rows, tops = [], []
    rng = np.random.default_rng(4)
    for n in ends:
        nxt = np.flatnonzero(v == v[n + 1])                   # the group that the next step of top_p adds
        tail = np.concatenate([[n], nxt])
        row = v[np.concatenate([rng.permutation(np.setdiff1d(np.arange(V), tail)), tail])]
        bits = np.float32(c[n]).view(np.uint32).astype(np.int64) + np.arange(-steps, steps + 1)
        tops.append(bits.astype(np.uint32).view(np.float32))
        rows += [row] * len(bits)
    tops = np.concatenate(tops)
    B = len(tops)
    t = lambda a: torch.as_tensor(a).cuda()
    off, temps = np.zeros(B + 1, np.int32), np.full(B, T, np.float32)
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    batch = fv.DeviceBatch(None, None, t(off), None, None, None, t(np.full(B, 1.0 - 2.0 ** -24, np.float32)), t(temps), None, None, None, 0,
                           None, off, temps)
    batch.top_p_host, batch.top_p = tops, t(tops)
    lg = torch.as_tensor(np.stack(rows)).to(torch.bfloat16).cuda()
    out = []
    for full in ("0", "1"):
        monkeypatch.setenv("FSV_NUCLEUS_FULL", full)
        res = fv.DeviceResult.alloc(B)
        ctx.sample(lg, batch, res)
        out.append(torch.stack([res.next_token, res.flags]).cpu().numpy())
    ctx.close()
    ids = out[1][0].reshape(8, -1)
    assert all(len(set(r.tolist())) > 1 for r in ids)         # every sweep crosses its edge
    assert (out[0] == out[1]).all(), int((out[0] != out[1]).any(0).sum())
