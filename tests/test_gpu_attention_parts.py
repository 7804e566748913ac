"""The attention kernel at the edges of its schedule: parts that end at and beside a multiple of eight key tiles, waves without a
tile, requests of one to three query-row tiles in one call, as many parts as it takes several batches to merge, and the
same launch again after one with other queries (the tickets a merge leaves must be those it found, and no partial result may be the other launch's)."""
import time

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_00644_amd import synth
from tests.helpers import logits_close
from tests.test_gpu_bf16_ops import _attention_case, _ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["mini64", "mini128"])
@pytest.mark.parametrize("seq_lens,gammas", [
    ([30, 31, 32, 223, 255, 256, 287], [0, 0, 7, 1, 0, 8, 16]),     # one part: one tile, two, seven, eight, nine
    ([511, 512, 1023, 1500, 20], [0, 16, 7, 8, 3]),                 # 16, 17, 32 tiles: two and more parts
    ([5000], [16]),                                                 # ten parts, three row tiles
    ([9000, 100, 4095], [1, 2, 7]),
    ([40 + 37 * i for i in range(100)], [i % 2 for i in range(100)]),        # two kv heads: four waves per block, one round
    ([3 + 61 * i % 997 for i in range(300)] + [7000], [7] * 300 + [1]),      # several rounds, long parts first
    ([511, 512, 480, 2047, 1000], [0, 0, 16, 0, 8]),                # 16 and 17 tiles, whole and cut; the longest call of one tile per wave
    ([511, 512, 480, 2048, 1000], [0, 0, 16, 0, 8]),                # and the next
    # row tiles that share their keys: two and three of them, four waves (head size 64: 192 pairs and more) and eight, one round and several
    ([30 + 37 * i for i in range(100)], [8 + i % 8 for i in range(100)]),
    ([25 + 29 * i for i in range(100)], [16 - i % 9 for i in range(100)]),
    ([20 + 53 * i for i in range(90)], [2 + 13 * (i % 3 > 0) for i in range(90)]),
    ([20 + 131 * i % 1999 for i in range(90)] + [9000], [16 - i % 2 for i in range(91)]),
])
def test_parts(name, seq_lens, gammas):
    ctx, batch, qd, check = _session(name, seq_lens, gammas)
    first = ctx.attention(1, qd, batch)
    assert not torch.equal(first, ctx.attention(0, -qd, batch))     # other queries: partial results that must not be met again
    assert torch.equal(first, ctx.attention(1, qd, batch))
    check(first)
    ctx.close()


@pytest.mark.parametrize("name", ["mini64", "mini128"])
def test_a_call_whose_lengths_disagree_spoils_no_later_one(name):
    """The device's lengths are those of shorter sessions than the host copies say (all pages stay within the table): the grid is
    larger than the schedule, the surplus blocks find empty records, and the next call is what it was."""
    ctx, batch, qd, check = _session(name, [5000, 3000, 800], [16, 3, 7])
    first = ctx.attention(1, qd, batch)
    lens = batch.seq_lens
    batch.seq_lens = torch.as_tensor(np.array([700, 300, 20], np.int32)).cuda()
    ctx.attention(1, qd, batch)
    batch.seq_lens = lens
    again = ctx.attention(1, qd, batch)
    assert torch.equal(first, again)
    check(again)
    ctx.close()


def test_the_schedule_of_many_long_requests_is_quickly_made():
    """300 requests of 32 k positions that all read the same pages: more (request, kv head) pairs than blocks, a length that no
    search for one round can find.  A call returns to its caller in well under the 3 ms that trying every part length took."""
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS["mini64"]
    B, L = 300, 32000
    pages = (L + 1 + 15) // 16
    _, ctx, w, wn = _ctx(cfg, 4, max_batch=B, max_gamma=1, max_pages=pages)
    kp, vp = fv.alloc_pools(cfg, pages)
    kp.zero_()
    vp.fill_(1.0)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()
    lens, off = np.full(B, L, np.int32), np.zeros(B + 1, np.int32)
    batch = fv.DeviceBatch(t(lens), None, t(off), None, None, None, None, None,
                           t(np.tile(np.arange(pages, dtype=np.int32), (B, 1))), kp, vp, pages, lens, off)
    q = torch.randn((B, cfg.n_heads, cfg.head_dim), generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    took = []
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        out = ctx.attention(1, q, batch)
        took.append(time.perf_counter() - t0)
    assert (out == 1.0).all()       # every value is one
    assert min(took) < 1e-3, took
    ctx.close()


def _session(name, seq_lens, gammas):
    cfg = synth.MODELS[name]
    L, gm, off, pt, npages, q, ks, vs = _attention_case(cfg, 8, seq_lens, gammas, "permuted")
    fv, ctx, w, wn = _ctx(cfg, 4, max_batch=len(L), max_gamma=16, max_pages=pt.shape[1])
    kp, vp = fv.alloc_pools(cfg, npages)
    kp.fill_(float("nan"))      # slots no position was written to
    vp.fill_(float("nan"))
    ptd = torch.as_tensor(pt).cuda()
    for b in range(len(L)):
        k = ks[b].expand(cfg.n_layers, -1, -1, -1).contiguous().cuda()
        v = vs[b].expand(cfg.n_layers, -1, -1, -1).contiguous().cuda()
        ctx.kv_import(kp, vp, npages, ptd[b], 0, k, v)
    batch = fv.DeviceBatch(torch.as_tensor(L).cuda(), None, torch.as_tensor(off).cuda(), None, None, None, None, None,
                           ptd, kp, vp, npages, L, off)

    def check(first):
        out = first.cpu().numpy().astype(np.float64)
        for b in range(len(L)):
            rs, n = int(off[b]) + b, int(gm[b]) + 1
            ref = oracle.attention(q[rs:rs + n].float().numpy(), ks[b][0].float().numpy(), vs[b][0].float().numpy(), int(L[b]))
            # the result is stored in fp16 (2^-11), its operands are exact to 2^-16
            ok, ratio = logits_close(out[rs:rs + n], ref, 2e-3)
            assert ok, (b, ratio)

    return ctx, batch, q.cuda(), check
