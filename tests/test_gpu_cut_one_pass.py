"""fp32 calls whose sampled requests all have a small top-k skip the row statistics (k_cut works from a sample's maximum): the same
result as with them, which FSV_NUCLEUS_FULL=1 brings back, for rows that the list settles and rows that it does not (ties, NaN,
infinities, too few finite logits), rows whose maximum the sample misses, greedy rows among them, and vocabularies around one
whole round of loads (32768)."""
import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth
from tests.test_gpu_cut import _laws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [32767, 32768, 32772, 50257, 98304, 100004])
@pytest.mark.parametrize("kind", ["normal", "flat", "ties", "peaked", "holes", "late", "infinite", "offset"])
def test_without_statistics(kind, V, monkeypatch):
    from paper_2601_00644_amd import flexverify as fv
    B, gam = 6, 2
    off = (np.arange(B + 1) * gam).astype(np.int32)
    g = torch.Generator().manual_seed(V)
    M = B * (gam + 1)
    if kind in ("late", "infinite", "offset"):
        z = torch.randn((M, V), generator=g) * 3.0
        if kind == "late":        # the sample is the first 8192 ids of each quarter of the whole rounds
            z[:, V - 1] = 30.0
            z[:, V - 2] = 29.5
        elif kind == "infinite":
            z[2, V - 1] = float("inf")
            z[4, 9] = float("inf")
            z[7, :] = -float("inf")
        else:
            z += 1000.0
    else:
        z = _laws(kind, M, V, g)
    lg = z.cuda()
    q = torch.softmax(torch.randn((B * gam, V), generator=g), -1).cuda()
    T = np.array([0.7, 1.0, 1.3, 0.0, 0.5, 1.0], np.float32)
    t = lambda a: torch.as_tensor(a).cuda()
    rng = np.random.default_rng(V)
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    d = rng.integers(0, V, B * gam).astype(np.int32)
    d[::2] = lg[torch.arange(0, M, 3).cuda()].nan_to_num(nan=-9e9).argmax(-1).cpu().numpy()     # first drafts: likely tokens
    batch = fv.DeviceBatch(None, None, t(off), t(d), q, t(synth.uniforms24(B * gam, V, 1)), t(synth.uniforms24(B, V, 2)), t(T), None,
                           None, None, 0, None, off, T)
    for top_k, top_p in (([1, 50, 341, 5, 2, 40], None), ([50] * B, [0.9, 1.0, 0.3, 0.9, 0.95, 0.999])):
        batch.top_k_host = np.asarray(top_k, np.int32)
        batch.top_k = t(batch.top_k_host)
        batch.top_p_host = None if top_p is None else np.asarray(top_p, np.float32)
        batch.top_p = None if top_p is None else t(batch.top_p_host)
        out = []
        for full in ("0", "1"):
            monkeypatch.setenv("FSV_NUCLEUS_FULL", full)
            res = fv.DeviceResult.alloc(B)
            ctx.sample(lg, batch, res)
            out.append(torch.stack([res.accepted_len, res.next_token, res.flags]).cpu().numpy())
        assert (out[0] == out[1]).all(), top_k
    ctx.close()


@pytest.mark.parametrize("sampled", [60, 59])
def test_more_rows_than_compute_units(sampled, monkeypatch):
    """270 rows: two thirds of them sampled, which leaves the statistics to k_cut, and one request less, which does not."""
    from paper_2601_00644_amd import flexverify as fv
    B, gam, V = 90, 2, 32772
    off = (np.arange(B + 1) * gam).astype(np.int32)
    g = torch.Generator().manual_seed(7)
    lg = (torch.randn((B * (gam + 1), V), generator=g) * 3.0).cuda()
    q = torch.softmax(torch.randn((B * gam, V), generator=g), -1).cuda()
    T = np.zeros(B, np.float32)
    T[np.random.default_rng(3).permutation(B)[:sampled]] = 0.8
    t = lambda a: torch.as_tensor(a).cuda()
    d = np.random.default_rng(5).integers(0, V, B * gam).astype(np.int32)
    d[::2] = lg[::gam + 1].argmax(-1).cpu().numpy()     # first drafts: likely tokens
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    batch = fv.DeviceBatch(None, None, t(off), t(d), q, t(synth.uniforms24(B * gam, V, 1)), t(synth.uniforms24(B, V, 2)), t(T), None,
                           None, None, 0, None, off, T)
    batch.top_k_host, batch.top_p_host = np.full(B, 50, np.int32), np.full(B, 0.9, np.float32)
    batch.top_k, batch.top_p = t(batch.top_k_host), t(batch.top_p_host)
    out = []
    for full in ("0", "1"):
        monkeypatch.setenv("FSV_NUCLEUS_FULL", full)
        res = fv.DeviceResult.alloc(B)
        ctx.sample(lg, batch, res)
        out.append(torch.stack([res.accepted_len, res.next_token, res.flags]).cpu().numpy())
    assert (out[0] == out[1]).all()
    assert 0 < out[0][0].sum() < B * gam
    ctx.close()
