"""Calls of up to 16 rows, whose projections carry the normalisation, the rotation, the append and the residual sum (few_rows.hip): one layer
against the oracle at the edges of its row counts and of the blocks its rules choose, and on the first row count past it.

Bars as everywhere: logits within 2e-2 of the fp64 oracle, layer-0 cache rows against the oracle with the bf16 storage points rounded.
"""
import numpy as np
import pytest
import torch

from paper_2601_00644_amd import synth
from tests.helpers import STORED_BF16, check_bf16_kv, check_bf16_logits
from tests.test_gpu_prefill import _oracle, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,kv_heads,hd,ffn,sessions", [
    (256, 4, 1, 64, 256, [(7, 1)]),                  # one row; shares of one step, the second half of a pair empty
    (256, 4, 2, 128, 768, [(15, 8)]),                # eight rows; shares of three steps
    (768, 6, 3, 128, 512, [(15, 2), (30, 7)]),       # nine rows of two requests; three steps of the normalised rows
    (256, 64, 16, 64, 8192, [(9, 5)]),               # q|k|v in pairs of tiles, gate|up in fours
    (256, 64, 16, 128, 512, [(20, 13)]),             # q|k|v in fours
    (256, 128, 32, 128, 256, [(9, 5)]),              # and in sevens
    (256, 4, 4, 64, 14336, [(0, 8)]),                # gate|up in sevens, 56 steps in down
    (256, 4, 4, 64, 14336, [(0, 16)]),               # sixteen rows and an ffn too long for the width: the kernels of more rows
    (1280, 4, 4, 64, 8448, [(0, 16)]),               # gate|up in sevens, sixteen rows, five steps of the normalised rows
    (2304, 4, 2, 64, 256, [(40, 11)]),               # more than eight steps a wave
    (2048, 4, 2, 64, 768, [(40, 7)]),                # o and down in tiles of eight features, the most blocks of them
    (2304, 4, 2, 64, 768, [(40, 7)]),                # and in tiles of sixteen, the fewest
    (3840, 4, 2, 128, 512, [(11, 2), (3, 6)]),
    (4096, 4, 1, 128, 14336, [(33, 3), (2, 5)]),     # the widest row, whole tiles added, eight rows
    (4096, 4, 1, 128, 512, [(3, 16)]),               # and sixteen
    (4096, 32, 8, 128, 8448, [(33, 3), (2, 5)]),     # the widest row, q|k|v in pairs of tiles and gate|up in sevens: eight rows
    (4096, 32, 8, 128, 8448, [(3, 16)]),             # and sixteen
    (256, 4, 4, 64, 256, [(0, 17)]),                 # seventeen rows: the kernels of more rows
])
def test_one_layer_matches_the_oracle(monkeypatch, d, heads, kv_heads, hd, ffn, sessions):
    name = f"few_{d}_{heads}_{kv_heads}_{hd}_{ffn}"
    monkeypatch.setitem(synth.MODELS, name, synth.ModelCfg(name, 1, d, heads, kv_heads, hd, ffn, 640, "bf16", 500000.0))
    fv, cfg, wn, chunks, ctxs, ctx, kp, vp, pt, page_rows, num_pages = _setup(name, sessions, 5, 15)
    batch = fv.prefill_pieces(chunks, page_rows, kp, vp, num_pages, 16)
    lg = ctx.prefill(batch, want_logits=True)
    again = ctx.prefill(batch, want_logits=True)
    assert torch.equal(lg, again)
    lg = lg.cpu().numpy().astype(np.float64)
    row = 0
    for (s_, L0, tokens), (r64, _, _), (rst, kst, vst) in zip(chunks, _oracle(cfg, wn, ctxs, chunks, 0), _oracle(cfg, wn, ctxs, chunks, STORED_BF16)):
        n = len(tokens)
        check_bf16_logits(lg[row:row + n], r64, rst, f"{name} session {s_}")
        row += n
        gk, gv = ctx.kv_export(kp, vp, num_pages, pt[s_], L0, n)
        for nm, got, want in (("k", gk, kst[:, L0:L0 + n]), ("v", gv, vst[:, L0:L0 + n])):
            check_bf16_kv(got.float().cpu().numpy().astype(np.float64).reshape(1, n, -1), want.reshape(1, n, -1), True, (s_, nm))
    ctx.close()


@pytest.mark.parametrize("d,ffn,rows,few", [
    (256, 4096, 16, True), (256, 4352, 8, True), (256, 4352, 9, False), (768, 8192, 9, True), (768, 8448, 9, False),
    (2048, 512, 16, True), (2304, 512, 8, True), (2304, 512, 9, False), (3840, 512, 16, False),
    (4096, 512, 8, True), (4096, 14336, 16, True), (4096, 14592, 8, True), (4096, 14592, 9, False),
    (2048, 512, 17, False),
])
def test_which_calls_take_the_layers_of_few_rows(monkeypatch, d, ffn, rows, few):
    """The rotation is a launch of its own where the layers of more rows are taken: from nine rows at widths whose normalisation costs more
    than the launches it saves."""
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.ModelCfg("route", 1, d, 4, 2, 64, ffn, 256, "bf16", 500000.0)
    ctx = fv.Context(cfg, synth.make_weights(cfg, 1, device="cuda"), max_batch=1, max_gamma=16, max_pages_per_req=2)
    kp, vp = fv.alloc_pools(cfg, 2)
    batch = fv.prefill_pieces([(0, 0, np.arange(rows, dtype=np.int32))], np.array([[0, 1]], np.int32), kp, vp, 2, 17)
    ctx.profile_enable(True)
    ctx.prefill(batch)
    launched = ctx.profile_read()
    assert ("rope_append" not in launched) == few, sorted(launched)
    ctx.close()
