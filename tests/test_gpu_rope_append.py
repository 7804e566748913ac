"""Rotation and KV append: value features handed to the threads in steps (at most two K slices) or in runs (more), against the oracle's
cache rows.  Head counts that leave a wave with keys and values, page boundaries inside a chunk, rows that are no multiple of eight.

Bar: layer-0 rows against the oracle with the bf16 storage points rounded, as everywhere (check_bf16_kv).
"""
import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth
from tests.helpers import STORED_BF16, check_bf16_kv
from tests.test_gpu_prefill import _oracle, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,kv_heads,hd,sessions", [
    (256, 4, 1, 64, [(7, 1)]),                 # one row
    (256, 8, 8, 64, [(15, 2), (30, 9)]),       # every head its own keys
    (256, 6, 3, 128, [(0, 17), (13, 20)]),     # 144 threads of q|k|v: waves with query, key and value heads
    (256, 12, 3, 64, [(0, 19)]),
    (1024, 6, 3, 128, [(5, 21)]),              # more than two slices: runs
    (512, 6, 3, 128, [(0, 130), (40, 141)]),   # more than 256 rows: the many-row product, one or two slices
])
def test_appended_rows_in_both_thread_orders(monkeypatch, d, heads, kv_heads, hd, sessions):
    name = f"append_{d}_{heads}_{kv_heads}_{hd}"
    monkeypatch.setitem(synth.MODELS, name, synth.ModelCfg(name, 1, d, heads, kv_heads, hd, 512, 640, "bf16", 500000.0))
    _, cfg, wn, chunks, ctxs, ctx, kp, vp, pt, page_rows, num_pages = _setup(name, sessions, 5, 15)
    from paper_2601_00644_amd import flexverify as fv
    ctx.prefill(fv.prefill_pieces(chunks, page_rows, kp, vp, num_pages, 16))
    torch.cuda.synchronize()
    for (s_, L0, tokens), (_, kst, vst) in zip(chunks, _oracle(cfg, wn, ctxs, chunks, STORED_BF16)):
        n = len(tokens)
        gk, gv = ctx.kv_export(kp, vp, num_pages, pt[s_], L0, n)
        for nm, got, want in (("k", gk, kst[:, L0:L0 + n]), ("v", gv, vst[:, L0:L0 + n])):
            check_bf16_kv(got.float().cpu().numpy().astype(np.float64).reshape(1, n, -1), want.reshape(1, n, -1), True, (s_, nm))
    ctx.close()
