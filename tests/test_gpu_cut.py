"""The top-k / top-p cut kernel (fsv_sample) where its fast way can go wrong, against the digit-by-digit way forced with
FSV_NUCLEUS_FULL=1: vocabularies around the rounds of its loads, ragged and unaligned rows, cuts of every depth, laws whose
candidates overflow its list, rows with -inf and NaN.  Both ways form the same integer masses; the windowed pass over bf16
logits measures top_p against the statistics' normaliser, which can move a cut only where the call flags it (bit 3)."""
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


def _cut_rank(v, T, top_k, top_p):
    """(tokens kept, least distance of the kept mass from top_p) by the definition, in fp64: v the logits in descending order."""
    e = np.exp((v.astype(np.float64) - float(v[0])) / float(T))
    n = len(v)
    if top_k:
        n = int(np.searchsorted(-v, -v[top_k - 1], side="right"))
    if top_p is None:
        return n, 1.0
    c = np.cumsum(e[:n]) / e[:n].sum()
    ends = np.flatnonzero(np.append(v[1:n] != v[:n - 1], True))       # last token of each group of equal logits
    at = int(np.searchsorted(c[ends], float(top_p)))
    lo = c[ends[at - 1]] if at else 0.0
    return int(ends[at]) + 1, min(float(top_p) - lo, float(c[ends[at]]) - float(top_p))


def _between(v, T, top_k, rank):
    """A top_p that falls half way into the mass of the group of equal logits that holds `rank`."""
    e = np.exp((v.astype(np.float64) - float(v[0])) / float(T))
    n = int(np.searchsorted(-v, -v[top_k - 1], side="right")) if top_k else len(v)
    a, b = np.searchsorted(-v[:n], -v[rank]), np.searchsorted(-v[:n], -v[rank], side="right")
    c = np.cumsum(e[:n]) / e[:n].sum()
    return np.float32(0.5 * ((c[a - 1] if a else 0.0) + c[b - 1]))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [64, 8191, 32768, 98312, 100003])
@pytest.mark.parametrize("law,T", [("normal", 0.7), ("normal", 1.0), ("normal", 3.0), ("offset", 0.8), ("flat", 1.0), ("ties", 0.8), ("nans", 1.0)])
def test_last_token_kept(law, T, V, dtype):
    """The cut itself: the id V - 2 holds the last token kept, V - 3 the one before it, V - 1 the first one cut, the others lie
    anywhere, and with u = 1 - 2^-24 the emitted id is the last one that has mass.  One token too many or too few emits another."""
    from paper_2601_00644_amd import flexverify as fv
    g = torch.Generator().manual_seed(V + len(law))
    z = torch.randn(V, generator=g)
    z = {"normal": z * 3.0, "offset": z * 3.0 + 20.0, "flat": z * 1e-2, "ties": (z * 2.0).round(), "nans": z * 3.0}[law].to(dtype)
    nans = np.full(5 if law == "nans" else 0, np.nan, np.float32)      # neither tokens nor mass
    v = z.float()[len(nans):].sort(descending=True).values.numpy()
    cuts = [(k, None) for k in (1, 2, 50, 341, 342, 1000, 2047, 2048, 2049, V // 2, V - 1) if k < len(v)]
    cuts += [(0, _between(v, T, 0, r)) for r in (0, 1, 60, 900, 2500, V // 3) if r < len(v)]
    cuts += [(k, _between(v, T, k, r)) for k, r in ((50, 0), (50, 20), (1000, 700), (2500, 1800), (30000, 20000)) if k < len(v)]
    e = np.exp((v.astype(np.float64) - float(v[0])) / T)
    rng, rows, used = np.random.default_rng(V), [], []
    for k, p in cuts:
        if p is not None and not 0.0 < p < 1.0:
            continue
        n, margin = _cut_rank(v, np.float32(T), k, p)
        # the draw has to be able to tell: a margin well above the masses' fixed point, the last token's mass above 2^-23 of the
        # whole, a token beyond the cut to emit by mistake
        if margin < 1e-6 or n >= len(v) - 1 or n < 3 or e[n - 1] < 2.0 ** -23 * e[:n].sum():
            continue
        tail = [n - 2, n - 1, n]
        rest = rng.permutation(np.concatenate([v[np.setdiff1d(np.arange(len(v)), tail)], nans]))
        rows.append(np.concatenate([rest, v[tail]]))
        used.append((k, p))
    B = len(rows)
    assert B >= 4
    t = lambda a: torch.as_tensor(a).cuda()
    off = np.zeros(B + 1, np.int32)
    temps = np.full(B, T, np.float32)
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    batch = fv.DeviceBatch(None, None, t(off), None, None, None, t(np.full(B, 1.0 - 2.0 ** -24, np.float32)), t(temps), None, None, None, 0,
                           None, off, temps)
    batch.top_k_host = np.array([k for k, _ in used], np.int32)
    batch.top_p_host = np.array([1.0 if p is None else p for _, p in used], np.float32)
    batch.top_k, batch.top_p = t(batch.top_k_host), t(batch.top_p_host)
    res = fv.DeviceResult.alloc(B)
    lg = torch.as_tensor(np.stack(rows)).to(dtype).cuda()
    if dtype == torch.bfloat16:
        lg.view(torch.int16)[lg.isnan()] = 0x7FC0      # (the conversion makes them negative, at the lower end of the key order)
    ctx.sample(lg, batch, res)
    got = res.next_token.cpu().numpy().tolist()
    ctx.close()
    assert got == [V - 2] * B, [(u, a) for u, a in zip(used, got) if a != V - 2]


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
