"""What the bf16 attention launches ask for in LDS, static words included, against what a compute unit has, for every list
length that the entry points accept.  On the CPU: the sizes come from the header that the launches use, compiled with the
host compiler, and the static ones from the assembly that the build keeps."""
import os
import re
import subprocess

from paper_2605_19726_amd import build
from test_compiled_waits import _asm_files

LDS = 160 * 1024
PROGRAM = r"""
#include <cstdio>
#include "attn_lds.hpp"
using namespace basa;
template <int D>
void table() {
  for (int nk = 1; nk <= (int)kMostBlocks<D>; ++nk) {
    std::printf("%d %d %zu", D, nk, most_lds<D>(nk));
    std::printf(" %zu", lds_bytes<D>(512, 32, nk));
    std::printf(" %zu", lds_bytes<D>(256, 32, nk));
    for (int causal = 0; causal < 2; ++causal)
      for (int fast = 0; fast < 2; ++fast)
        std::printf(" %zu", lds_bytes<D>(512, 64, nk, causal, fast, launch_stages<D>(512, 64, nk, causal, fast)));
    std::printf("\n");
  }
}
int main() { table<64>(); table<128>(); }
"""


def _static():
    """{(queries per workgroup, without running maxima): static LDS bytes} over the attention kernels of the build."""
    (path,) = [f for f in _asm_files() if os.path.basename(f).startswith("attn_mfma-")]
    most, kernel = {}, None
    for line in open(path):
        m = re.match(r"\s*\.amdhsa_kernel (\S+)", line)
        if m:
            one = re.search(r"attn_mfma_kernelILi\d+ELi\d+ELi(\d+)ELi\d+ELb\dELb(\d)", m.group(1))
            many = re.search(r"(Attn|Wide)JobILi\d+ELi\d+E(?:Lb(\d))?", m.group(1))
            rows = re.search(r"attn_rows_kernelILi\d+ELi\d+ELb(\d)", m.group(1))
            kernel = (int(one.group(1)), one.group(2) == "1") if one else (128, rows.group(1) == "1") if rows else \
                     (512 if many.group(1) == "Wide" else 128, many.group(2) != "0") if many else None
        m = re.match(r"\s*\.amdhsa_group_segment_fixed_size (\d+)", line)
        if m and kernel:
            most[kernel] = max(most.get(kernel, 0), int(m.group(1)))
    return most


def test_no_accepted_call_asks_for_more_lds_than_there_is(tmp_path):
    static = _static()
    assert set(static) == {(512, True), (512, False), (256, False), (128, True), (128, False)}
    (tmp_path / "t.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")], check=True)
    rows = subprocess.run([str(tmp_path / "t")], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    accepted = {64: 0, 128: 0}
    for row in rows:
        d, nk, most, shared, solo, plain, fast, c_plain, c_fast = map(int, row.split())
        real = max(shared + static[256, False], solo + static[128, True], plain + static[512, False], fast + static[512, True],
                   c_plain + static[512, False], c_fast + static[512, True])
        assert most >= real, (d, nk, most, real)          # (what the entry points refuse by)
        if shared + static[256, False] <= LDS:            # a call that the two-stage rings have room for is not refused
            assert most <= LDS, (d, nk, most)
            accepted[d] = nk
    assert accepted == {64: 8192, 128: 8184}
