"""When the 128-query attention shape reads the rows of K and V itself, on both sides of the lines that were measured and of the limits
of its arithmetic.  On the CPU: the rules stand in a header of plain C++, compiled here with the host compiler."""
import subprocess

import pytest

from paper_2605_19726_amd import build

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "attn_rows.hpp"
int main(int argc, char** argv) {
  const bool yes = argc == 4 ? basa::rows_pay((size_t)std::atoll(argv[1]), std::atof(argv[2]), std::atoi(argv[3]) != 0)
                             : basa::offsets_fit(std::atoll(argv[1]), std::atoll(argv[2]));
  std::printf("%d\n", yes ? 1 : 0);
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    (d / "r.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(d / "r.cpp"), "-o", str(d / "r")], check=True)
    return lambda *args: subprocess.run([str(d / "r"), *map(str, args)], check=True, capture_output=True, text=True).stdout == "1\n"


# bytes of K, estimate of the attention, d = 64 and a compute unit to each whole list
@pytest.mark.parametrize("heads_kv,L,d,us,alone,rows", [
    (8, 32768, 128, 50.0, False, True), (8, 4000, 128, 20.0, False, True), (8, 8000, 128, 170.0, False, True), (2, 8000, 128, 150.0, False, False),
    (8, 4000, 128, 128.0, False, False), (2, 640, 64, 14.7, True, True), (2, 1216, 64, 22.1, True, False), (2, 3200, 64, 40.7, True, False),
    (1, 2496, 64, 34.2, True, False), (8, 2496, 64, 34.2, True, False), (8, 1280, 64, 17.9, True, True), (8, 2432, 64, 34.0, False, True)])
def test_calls_read_rows_where_that_measured_faster(ask, heads_kv, L, d, us, alone, rows):
    assert ask(heads_kv * L * d * 2, us, int(alone)) == rows


@pytest.mark.parametrize("L,stride,fit", [
    (1, 64, True), (32768, 128, True), (1, 2 ** 23 - 8, True), (1, 2 ** 23, False), (2 ** 24 - 1, 64, True), (2 ** 24, 64, False),
    (2 ** 24 - 1, 120, True), (2 ** 24 - 1, 136, False), (2 ** 16, 2 ** 15 - 8, True), (2 ** 16, 2 ** 15, False), (256, 2 ** 23 - 8, True), (257, 2 ** 23 - 8, False)])
def test_offsets_of_rows_fit_24_by_24_bits_in_32(ask, L, stride, fit):
    assert ask(L, stride) == fit
    # the last byte that a lane addresses, from the first of the head: no wrap, and no factor past 24 bits
    assert not fit or (2 * stride < 2 ** 24 and L - 1 < 2 ** 24 and (L - 1) * 2 * stride + 256 <= 2 ** 32)
