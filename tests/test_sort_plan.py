"""Tiles that a norm sort starts from, on both sides of the lines that were measured.  On the CPU: the rule stands in a header
of plain C++, compiled here with the host compiler."""
import subprocess

import pytest

from paper_2605_19726_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "sort_plan.hpp"
int main(int argc, char** argv) {
  long v[7];
  for (int i = 0; i < 7; ++i) v[i] = std::atol(argv[i + 1]);
  const basa::SortPlan p = basa::plan_sort(v[0], (int)v[1], v[2], (int)v[3], (int)v[4], (int)v[5], v[6] != 0);
  std::printf("%d %d\n", p.few ? 1 : 0, p.tile);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(d / "p.cpp"), "-o", str(d / "p")], check=True)

    def call(rows0, L0, rows1=0, L1=0, window=0, token_bytes=256, cached=True):
        args = [str(int(x)) for x in (rows0, L0, rows1, L1, window, token_bytes, cached)]
        few, tile = subprocess.run([str(d / "p"), *args], check=True, capture_output=True, text=True).stdout.split()
        return few == "1", int(tile)
    return call


# runs that leave most of a quad of 16384 words empty: one tile of 4096, or two and a merge pass, is the whole run
@pytest.mark.parametrize("rows,L,window,tile", [
    (1024, 1024, 0, 1024), (699, 1500, 0, 1024), (300, 2048, 0, 1024), (300, 2049, 0, 4096), (350, 3000, 0, 4096), (256, 4096, 0, 4096),
    (512, 4096, 0, 4096), (128, 5000, 0, 4096), (130, 5000, 0, 1024), (256, 5000, 0, 1024), (258, 5000, 0, 4096), (128, 8192, 0, 4096),
    (130, 8192, 0, 1024), (160, 8192, 0, 1024), (162, 8192, 0, 4096), (64, 8193, 0, 1024), (96, 8300, 0, 1024), (64, 32768, 0, 1024),
    (65, 32768, 0, 4096), (32, 32768, 1024, 1024), (32, 32768, 2048, 1024), (32, 32768, 4096, 4096), (32, 32768, 8192, 4096),
    (34, 32768, 8192, 1024), (32, 32768, 16384, 1024), (600, 1000, 4096, 1024)])
def test_middling_calls_start_from_the_tiles_that_fill_a_quad(plan, rows, L, window, tile):
    assert plan(rows, L, window=window) == (False, tile)
    assert plan(rows, L, window=window, cached=False) == (False, tile)
    if rows % 2 == 0:
        assert plan(rows // 2, L, rows // 2, L, window=window) == (False, tile)


# one head's rows are read by twice as many workgroups, which has to leave them at one to a compute unit (more where the second
# large tile of a run is hardly used, and with short tokens)
@pytest.mark.parametrize("rows,L,window,token_bytes,tile", [
    (1, 1024, 0, 256, 1024), (1, 1025, 0, 256, 512), (1, 4096, 0, 256, 512), (1, 4097, 0, 256, 1024), (32, 4096, 0, 256, 512),
    (33, 4096, 0, 256, 1024), (128, 4096, 0, 256, 1024), (42, 3000, 0, 256, 512), (44, 3000, 0, 512, 1024), (341, 1536, 0, 256, 512),
    (100, 2048, 0, 256, 512), (101, 2048, 0, 256, 1024), (80, 4096, 0, 128, 512), (81, 4096, 0, 128, 1024), (256, 2048, 0, 128, 512),
    (32, 8192, 4096, 256, 1024), (16, 8192, 4096, 256, 512), (8, 60000, 1024, 256, 1024)])
def test_calls_of_few_words_start_from_512_tokens_while_the_device_has_room(plan, rows, L, window, token_bytes, tile):
    assert plan(rows, L, window=window, token_bytes=token_bytes) == (True, tile)
    assert plan(rows, L, window=window, token_bytes=token_bytes, cached=False) == (True, 1024)
    if rows > 1:
        assert plan(rows - 1, L, 1, L, window=window, token_bytes=token_bytes) == (True, tile)
