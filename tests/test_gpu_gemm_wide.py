"""The many-row projection kernel at the edges of its blocks (64 MT rows x 256 features), of the K cut and of the strip count,
forced with FSV_GEMM_WIDE: single projections against the oracle, the whole forward (SwiGLU and logits epilogues) against
the weight-streaming kernel."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2601_00644_amd import synth
from tests.helpers import logits_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [2, 3, 4])
@pytest.mark.parametrize("name,M", [("mini64", 1), ("mini64", 64), ("mini64", 65), ("mini128", 127), ("mini64", 129), ("mini128", 193),
                                    ("mini64", 256), ("mini128", 257), ("mini64", 449)])
def test_linear_matches_oracle(name, M, tiles, monkeypatch):
    from paper_2601_00644_amd import flexverify as fv
    monkeypatch.setenv("FSV_GEMM_WIDE", str(tiles))
    cfg = synth.MODELS[name]        # 256 .. 1536 contraction elements, 97 and 157 strips in the head
    w = synth.make_weights(cfg, 3, std=0.05)
    ctx = fv.Context(cfg, {k: v.cuda() for k, v in w.items()}, 8, 16, 4, max_rows=max(M, 136))
    g = torch.Generator().manual_seed(10 * M + tiles)
    for wh, key, K in [(fv.W_QKV, "w_qkv.1", cfg.d_model), (fv.W_O, "w_o.0", cfg.n_heads * cfg.head_dim),
                       (fv.W_GATE_UP, "w_gate_up.1", cfg.d_model), (fv.W_DOWN, "w_down.0", cfg.d_ffn), (fv.W_LM_HEAD, "lm_head", cfg.d_model)]:
        x = torch.randn((M, K), generator=g).to(torch.bfloat16)
        wt = w[key].view(torch.int16).numpy().view(np.uint16)
        y = ctx.linear(wh, int(key.split(".")[1]) if "." in key else 0, x.cuda(), wt.shape[0]).cpu().numpy().astype(np.float64)
        # exact 16-bit products summed in fp32: the bar of the weight-streaming kernel's own test
        ok, ratio = logits_close(y, oracle.linear(wt, x.float().numpy().astype(np.float64), True), 1e-3)
        assert ok, (key, M, ratio)
    ctx.close()


@pytest.mark.parametrize("tiles", [2, 3, 4])
@pytest.mark.parametrize("name,rows", [("mini128", 33), ("mini64", 290)])
def test_forward_matches_the_weight_streaming_kernel(name, rows, tiles, monkeypatch):
    from paper_2601_00644_amd import flexverify as fv
    cfg = synth.MODELS[name]
    w = {k: v.cuda() for k, v in synth.make_weights(cfg, 5, std=0.04).items()}
    toks = np.random.default_rng(rows).integers(0, cfg.vocab, rows).astype(np.int32)
    mp = rows // 16 + 2
    page_rows = np.arange(mp, dtype=np.int32)[None, :]
    out = []
    for force in (0, tiles):
        monkeypatch.setenv("FSV_GEMM_WIDE", str(force))
        ctx = fv.Context(cfg, w, max_batch=rows // 16 + 1, max_gamma=15, max_pages_per_req=mp, max_rows=rows)
        kp, vp = fv.alloc_pools(cfg, mp)
        out.append(ctx.prefill(fv.prefill_pieces([(0, 0, toks)], page_rows, kp, vp, mp, 16), want_logits=True).cpu())
        ctx.close()
    # The two differ by the order of fp32 sums only.  Where that moves a 16-bit tensor between the kernels across a rounding
    # boundary, the forwards part as two correct 16-bit forwards do: by less than each is from fp64 (the 2e-2 bar).
    a, b = out
    assert ((a - b).norm(dim=1) <= 2e-2 * a.norm(dim=1)).all()
