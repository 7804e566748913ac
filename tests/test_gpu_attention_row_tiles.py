"""Attention schedules past the line up to which row tiles are parts of their own in any case: calls whose longest parts say split, and calls
beside them whose longest parts say shared (two kv heads, a few requests of two row tiles)."""
import pytest
import torch

from tests.test_gpu_attention_parts import _session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["mini64", "mini128"])
@pytest.mark.parametrize("seq_lens,gammas", [
    ([6900 + 37 * i for i in range(20)], [8 if i % 6 == 0 else i % 7 for i in range(20)]),     # longest parts 40 and 46 tiles: split
    ([7600 + 37 * i for i in range(20)], [8 if i % 6 == 0 else i % 7 for i in range(20)]),     # past 42 tiles: split with head size 64
    ([6900 + 37 * i for i in range(20)], [8 + i % 8 for i in range(20)]),                      # 50 and 78 tiles: shared with head size 128
])
def test_row_tiles_split_by_the_longest_part(name, seq_lens, gammas):
    ctx, batch, qd, check = _session(name, seq_lens, gammas)
    first = ctx.attention(1, qd, batch)
    assert torch.equal(first, ctx.attention(1, qd, batch))
    check(first)
    ctx.close()
