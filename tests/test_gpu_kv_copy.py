"""Session import / export (fsv_kv_import / fsv_kv_export, FSV_BF16): whole pages go through 16-byte units, partial pages and
unaligned arrays element by element.  Both against the element order the header documents, bit for bit."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth

pytestmark = pytest.mark.gpu


def _tile_order(hd):
    t, e = np.meshgrid(np.arange(16), np.arange(hd), indexing="ij")
    return ((e // 16 * 2 + (e % 16) // 8) * 16 + t) * 8 + e % 8, ((e // 32 * 2 + (t % 8) // 4) * 32 + e % 32) * 8 + 4 * (t // 8) + t % 4


def _shifted(x, by):
    """A contiguous copy of x whose storage starts `by` elements after an aligned address."""
    buf = torch.zeros(x.numel() + 8, dtype=x.dtype, device="cuda")
    y = buf[by:by + x.numel()].view(x.shape)
    y.copy_(x)
    return y


@pytest.mark.parametrize("name,heads,kv,pos0,n,shift", [
    ("mini128", 8, 2, 0, 16, 0),        # one whole page
    ("mini128", 8, 2, 0, 15, 0),        # one partial page
    ("mini128", 8, 2, 5, 6, 0),         # inside one page
    ("mini128", 8, 2, 3, 77, 0),        # partial, whole, partial
    ("mini128", 8, 8, 16, 64, 0),       # two head groups
    ("mini128", 10, 5, 7, 60, 0),       # a ragged head group
    ("mini128", 8, 1, 0, 48, 1),        # unaligned arrays
    ("mini64", 8, 2, 1, 50, 0),
    ("mini64", 20, 5, 0, 33, 0),
    ("mini64", 8, 8, 0, 112, 4),
])
def test_copy_follows_the_documented_tiles(name, heads, kv, pos0, n, shift):
    from paper_2601_00644_amd import flexverify as fv
    cfg = dataclasses.replace(synth.MODELS[name], n_heads=heads, n_kv_heads=kv)
    w = synth.make_weights(cfg, 3)
    pages = 9
    ctx = fv.Context(cfg, {k: t.cuda() for k, t in w.items()}, max_batch=1, max_gamma=1, max_pages_per_req=8)
    pt = torch.tensor([6, 0, 8, 3, 1, 7, 2, 4], dtype=torch.int32)
    k, v = synth.make_kv_context(cfg, n, 5, 0)
    kp, vp = fv.alloc_pools(cfg, pages)
    kp.fill_(7.0)
    vp.fill_(7.0)
    ctx.kv_import(kp, vp, pages, pt.cuda(), pos0, _shifted(k, shift), _shifted(v, shift))
    ko, vo = _tile_order(cfg.head_dim)
    for pool, src, order in ((kp, k, ko), (vp, v, vo)):
        want = torch.full((cfg.n_layers, pages, kv, 16 * cfg.head_dim), 7.0, dtype=torch.bfloat16)
        for i in range(n):
            pos = pos0 + i
            want[:, int(pt[pos // 16]), :, torch.as_tensor(order[pos % 16])] = src[:, i]
        assert torch.equal(pool.cpu(), want)      # in place, and nothing else written
    gk, gv = ctx.kv_export(kp, vp, pages, pt.cuda(), pos0, n)
    assert torch.equal(gk.cpu(), k) and torch.equal(gv.cpu(), v)
    ctx.close()
