"""Logits and draft laws whose rows lie at 2- and 4-byte boundaries (odd vocabularies, arrays that do not start at 16 bytes): what the
aligned copies give, with and without cuts."""
import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [9, 2047, 8192, 8195, 40001])
@pytest.mark.parametrize("top_k,top_p", [(0, 1.0), (0, 0.9), (7, 0.9)])
def test_any_boundary(V, dtype, top_k, top_p):
    from paper_2601_00644_amd import flexverify as fv
    B, gam = 5, 3
    off = (np.arange(B + 1) * gam).astype(np.int32)
    G, M = B * gam, B * gam + B
    g = torch.Generator().manual_seed(V)
    lg = (torch.randn((M, V), generator=g) * 3.0).to(dtype).cuda()
    q = torch.softmax(torch.randn((G, V), generator=g) * 3.0, -1).cuda()
    T = np.array([0.7, 1.0, 0.0, 0.5, 1.3], np.float32)
    t = lambda a: torch.as_tensor(a).cuda()
    d = torch.multinomial(q, 1).squeeze(1).to(torch.int32)
    ctx = fv.Context(synth.ModelCfg("sampler", 0, 0, 0, 0, 0, 0, V, "bf16"), None, B, 16, sampler_only=True)
    out = []
    for shift in (0, 1, 3):
        lbuf = torch.full((lg.numel() + 16,), float("nan"), dtype=dtype, device="cuda")
        qbuf = torch.full((q.numel() + 16,), float("nan"), device="cuda")
        ls, qs = lbuf[shift:shift + lg.numel()].view(M, V), qbuf[shift:shift + q.numel()].view(G, V)
        ls.copy_(lg)
        qs.copy_(q)
        batch = fv.DeviceBatch(None, None, t(off), d, qs, t(synth.uniforms24(G, V, 1)), t(synth.uniforms24(B, V, 2)), t(T), None, None,
                               None, 0, None, off, T)
        if top_p < 1.0:
            batch.top_p_host = np.full(B, top_p, np.float32)
            batch.top_p = t(batch.top_p_host)
        if top_k:
            batch.top_k_host = np.full(B, top_k, np.int32)
            batch.top_k = t(batch.top_k_host)
        res = fv.DeviceResult.alloc(B)
        ctx.sample(ls, batch, res)
        out.append(torch.stack([res.accepted_len, res.next_token, res.flags]).cpu().numpy())
    assert (out[0] == out[1]).all() and (out[0] == out[2]).all()
    assert (out[0][1] >= 0).all() and (out[0][1] < V).all()
    ctx.close()
