"""Blocks of one launch that hand results to the block drawing the last ticket: in the library's gfx950 code every wave waits for its
stores (vmcnt) before the barrier in front of the ticket.  Without that wait the ticket can be seen before the results, which no
comparison of outputs shows reliably, so the code itself is read (no GPU work)."""
import os
import re
import shutil
import subprocess

import pytest

from tests.test_library_exports import LIB, _lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
TICKET = re.compile(r"\s*global_atomic_add .* sc0\b")      # an add whose old value is used


def _kernels(tmp_path):
    """{mangled name: instructions in the order of the code} of every device function of the library."""
    _lib()
    so = shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", so], cwd=tmp_path, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                out[m.group(1)] = body = []
            elif line.startswith("\t"):
                body.append(line.split("//")[0].strip())
    return out


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs ROCm's llvm-objdump")
@pytest.mark.parametrize("kernel,instantiations", [("k_attention", 10), ("k_decide", 2)])
def test_stores_are_complete_before_the_ticket(tmp_path, kernel, instantiations):
    found = 0
    for name, code in _kernels(tmp_path).items():
        if kernel not in name:
            continue
        for at, ins in enumerate(code):
            if not TICKET.match(ins):
                continue
            found += 1
            barrier = max(i for i in range(at) if code[i] == "s_barrier")
            wait = max((i for i in range(barrier) if re.search(r"s_waitcnt .*\bvmcnt\(0\)", code[i])), default=-1)
            # the wait stands right before the barrier: no memory access and no branch in between
            between = code[wait + 1:barrier]
            assert wait >= 0 and not any(re.match(r"(global|flat|buffer|scratch)_|s_c?branch", i) for i in between), (name, between[:8])
    assert found == instantiations
