"""fsv_attention with query and result arrays at 2- and 4-byte boundaries (the query operand is packed in the set-up launch, the
result written as rows by the attention kernels): bit for bit what aligned arrays give, one part per request and several."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["mini64", "mini128"])
@pytest.mark.parametrize("L", [[0, 17, 3], [700, 40, 1500]])
def test_unaligned_arrays(name, L):
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS[name]
    gam = np.array([2, 0, 11], np.int32)
    L = np.asarray(L, np.int32)
    off = np.concatenate([[0], np.cumsum(gam)]).astype(np.int32)
    pt, n = synth.make_page_table(L, gam, 16, "permuted", 2)
    ctx = fv.Context(cfg, {k: v.cuda() for k, v in synth.make_weights(cfg, 1).items()}, max_batch=3, max_gamma=16,
                     max_pages_per_req=pt.shape[1])
    kp, vp = fv.alloc_pools(cfg, n)
    kp.normal_()
    vp.normal_()
    t = lambda a: torch.as_tensor(a).cuda()
    batch = fv.DeviceBatch(t(L), None, t(off), None, None, None, None, None, t(pt), kp, vp, n, L, off)
    M, w = batch.rows, cfg.n_heads * cfg.head_dim
    q = torch.randn((M, cfg.n_heads, cfg.head_dim), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
    want = ctx.attention(1, q, batch)
    buf = torch.empty(q.numel() + 8, dtype=torch.bfloat16, device="cuda")
    qs = buf[1:1 + q.numel()].view(q.shape)
    qs.copy_(q)
    res = torch.full((M * w + 9,), 7.0, device="cuda")
    b = batch.struct()
    rc = fv.lib().fsv_attention(ctx._h, 1, C.c_void_p(qs.data_ptr()), C.byref(b), C.c_void_p(res.data_ptr() + 4),
                                C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(res[1:1 + M * w].view(M, w), want)
    assert res[0] == 7.0 and (res[1 + M * w:] == 7.0).all()
    ctx.close()
