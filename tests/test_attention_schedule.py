"""Which attention schedule a call is given (csrc/attn_schedule.h, plain C++, compiled here without the GPU): the query-row tiles of a request
together, or as parts of their own, on both sides of every line of that rule (256 compute units).

Each case: the costs of the longest part of both schedules in 1/16 of a key tile, worked out by the driver, and which of the two is taken."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def schedule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("schedule") / "driver")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", os.path.join(HERE, "attn_schedule_main.cpp"), "-o", exe])

    def run(hd, kv_heads, group, requests):
        line = " ".join(str(v) for v in (hd, kv_heads, group, 256, len(requests), *(x for r in requests for x in r)))
        out = subprocess.run([exe], input=line.encode(), capture_output=True, timeout=60, check=True).stdout
        names = "rt nw tpw blocks split sorted together together_blocks together_sorted apart apart_blocks apart_sorted"
        return dict(zip(names.split(), map(int, out.split()), strict=True))
    return run


def _calls(n, first, step, drafts):
    return [(first + step * i, drafts[i % len(drafts)]) for i in range(n)]


@pytest.mark.parametrize("hd,call,together,apart,split", [
    # all (row tile, key tile) pairs come to four a wave, and one more than that (where the longest parts say the other thing)
    (64, (4, 4070, 0, (15,)), 320, 512, True), (64, (10, 1450, 37, (15,)), 360, 800, False),
    (128, (8, 2020, 0, (15,)), 320, 512, True), (128, (11, 1720, 37, (15, 7)), 448, 880, False),
    # the longest part of the shared schedule: up to 66 tiles (head size 64) and 42 (128), and the next
    (64, (9, 6330, 0, (8, 1)), 1056, 1600, True), (64, (19, 1410, 101, (15, 7)), 1072, 1536, False),
    (64, (8, 6740, 0, (15,)), 1060, 1696, False),
    (128, (5, 6620, 0, (8, 0)), 672, 832, True), (128, (9, 3190, 0, (8, 8, 3)), 680, 800, False),
    # its ratio to that of the other: from 0.625 (head size 64) and 0.7 (128)
    (64, (12, 1360, 101, (8, 1)), 500, 800, True), (64, (7, 4930, 101, (15,)), 820, 1344, False),
    (128, (3, 8940, 37, (15,)), 640, 912, True), (128, (3, 6690, 37, (15,)), 480, 688, False),
    # a row tile more than there are blocks for
    (64, (16, 790, 37, (15,)), 440, 688, True), (64, (17, 280, 0, (15,) * 16 + (0,)), None, None, False),
    (128, (16, 280, 0, (15,)), 200, 160, True),
    # one row tile in every request: nothing to split
    (128, (8, 2020, 0, (7,)), 256, 256, False),
])
def test_row_tiles_together_or_apart(schedule, hd, call, together, apart, split):
    p = schedule(hd, 8, 4, _calls(*call))
    if together is not None:
        assert (p["together"], p["apart"]) == (together, apart)
    assert p["split"] == split
    assert p["rt"] == (1 if split else max(-(-4 * (g + 1) // 32) for _, g in _calls(*call)))
    assert p["blocks"] == (p["apart_blocks"] if split else p["together_blocks"])


@pytest.mark.parametrize("hd,first,drafts,together,apart,split", [
    (64, 6900, lambda i: 8 if i % 6 == 0 else i % 7, 40, 46, True), (128, 6900, lambda i: 8 if i % 6 == 0 else i % 7, 40, 46, True),
    (64, 7600, lambda i: 8 if i % 6 == 0 else i % 7, 50, 51, True), (128, 7600, lambda i: 8 if i % 6 == 0 else i % 7, 50, 51, False),
    (64, 6900, lambda i: 8 + i % 8, 50, 78, True), (128, 6900, lambda i: 8 + i % 8, 50, 78, False),
])
def test_the_calls_compared_on_the_gpu_take_both(schedule, hd, first, drafts, together, apart, split):
    """The calls whose results tests/test_gpu_attention_row_tiles.py compares (two kv heads; costs in whole tiles)."""
    p = schedule(hd, 2, 4, [(first + 37 * i, drafts(i)) for i in range(20)])
    assert (p["together"] / 16, p["apart"] / 16, p["split"]) == (together, apart, split)
