"""Where the tile loop of the 512-query attention kernels starts in a line of 64 bytes: at the offsets that were measured as the fastest,
in every form that walks in spans.  On the CPU, on the code object that the build keeps in _build/."""
import os
import re
import subprocess

import pytest

from paper_2605_19726_amd import build
from test_compiled_waits import _asm_files

OBJDUMP = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin", "llvm-objdump")
if not os.path.exists(OBJDUMP):
    OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _loop_start(body):
    """Address of the first block of the innermost loop around a barrier and the products of a tile."""
    products, barriers, back = [], [], []
    for line in body:
        m = re.match(r"\s+(\S+)(.*)// ([0-9A-F]+)", line)
        if not m:
            continue
        at = int(m.group(3), 16)
        if m.group(1).startswith("v_mfma"):
            products.append(at)
        elif m.group(1) == "s_barrier":
            barriers.append(at)
        elif re.match(r"s_c?branch", m.group(1)):
            words = int(m.group(2).split()[0])
            to = at + 4 + 4 * (words - 65536 if words >= 32768 else words)
            if to < at:
                back.append((at - to, to, at))
    loops = [(size, a) for size, a, b in back if sum(a <= x <= b for x in products) >= 32 and any(a <= x <= b for x in barriers)]
    return min(loops)[1]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler for the objects of this build")
def test_tile_loops_start_where_they_were_measured():
    _asm_files()
    obj = os.path.join(build.OBJ_DIR, "attn_mfma-hip-amdgcn-amd-amdhsa-gfx950.out")
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
    form = re.compile(r"attn_mfma_kernelILi(64|128)ELi128ELi512ELi64ELb0ELb1ELb0E|WideJobILi(64|128)ELi128ELb1E")
    found = {}
    for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n((?:.+\n)*)", text, re.M):
        m = form.search(name)
        if m:
            found["call" if m.group(1) else "batch", int(m.group(1) or m.group(2))] = _loop_start(body.split("\n")) % 64
    assert found == {("call", 128): 56, ("batch", 128): 56, ("call", 64): 20, ("batch", 64): 20}
