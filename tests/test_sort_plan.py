"""Tiles that a norm sort starts from, on both sides of the lines that were measured, and the values at which its merge cuts their
runs.  On the CPU: the rules stand in a header of plain C++, compiled here with the host compiler."""
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


# runs of 2049 to 8192 tokens: one tile of 4096, or two and a merge pass, is the whole run, but for 129 to 256 of the longer ones
@pytest.mark.parametrize("rows,L,window,tile", [
    (1024, 1024, 0, 1024), (699, 1500, 0, 1024), (300, 2048, 0, 1024), (300, 2049, 0, 4096), (350, 3000, 0, 4096), (256, 4096, 0, 4096),
    (512, 4096, 0, 4096), (128, 5000, 0, 4096), (130, 5000, 0, 1024), (256, 5000, 0, 1024), (258, 5000, 0, 4096), (128, 8192, 0, 4096),
    (130, 8192, 0, 1024), (160, 8192, 0, 1024), (162, 8192, 0, 4096), (64, 8193, 0, 1024), (96, 8300, 0, 1024), (64, 32768, 0, 1024),
    (65, 32768, 0, 4096), (32, 32768, 1024, 1024), (32, 32768, 2048, 1024), (32, 32768, 4096, 4096), (32, 32768, 8192, 4096),
    (34, 32768, 8192, 1024), (32, 32768, 16384, 1024), (600, 1000, 4096, 1024)])
def test_middling_calls_start_from_the_tiles_of_their_run_length(plan, rows, L, window, tile):
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


CUTS = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "sort_plan.hpp"
using namespace basa;
// A group of `n` words in sorted runs of 1024, cut into parts of `samples` samples: every cut has exactly as many samples below it as
// asked for, in the steps of a search between two neighbouring samples, and no part exceeds what the kernel has room for.
int main(int argc, char** argv) {
  const int n = std::atoi(argv[1]), samples = std::atoi(argv[2]), kind = std::atoi(argv[3]);
  std::mt19937_64 rng(n + 7 * samples + kind);
  std::vector<uint64_t> w(n);
  for (int i = 0; i < n; ++i) {
    uint64_t key = 0x3f000000u + (rng() & 0xffffff);                     // 0: spread
    if (kind == 1) key = i >= n / 1024 * 1024 ? 0 : key;                 // short last run: zeros (padding tokens)
    if (kind == 2) key = i >= n / 1024 * 1024 ? 0x7f800000u : key;       // ... infinities
    if (kind == 3) key = 0x3f000000u;                                    // all alike
    if (kind == 4) key = 0x3f000000u + i;                                // ascending
    if (kind == 5) key = 0x3f000000u + n - i;                            // descending
    if (kind == 6) key = 0x3f000000u + i % 1024;                         // every run alike
    if (kind == 7) key = i >= n / 1024 * 1024 ? 0 : 0x3f000000u + i % 1024;
    w[i] = key << 27 | (uint64_t)i;
  }
  std::vector<uint64_t> all;
  const int runs = (n + kSmallTile - 1) / kSmallTile;
  for (int r = 0; r < runs; ++r) {
    std::sort(w.begin() + r * kSmallTile, w.begin() + std::min(n, (r + 1) * kSmallTile));
    for (int i = r * kSmallTile; i < std::min(n, (r + 1) * kSmallTile); i += kCutStride) all.push_back(w[i]);
  }
  int worst = 0;
  size_t words_before = 0;
  for (int want = samples; want * kCutStride < n; want += samples) {
    const CutBracket at = cut_bracket(want, n);
    if (at.highest > 15 || at.lowest > 15) return std::printf("sample %d, %d of a run\n", at.lowest, at.highest), 1;
    uint64_t lo = ~0ull, hi = 0;
    for (int r = 0; r < runs; ++r) {
      auto sample = [&](int k) { return r * kSmallTile + k * kCutStride; };
      if (sample(at.lowest) < n) lo = std::min(lo, w[sample(at.lowest)]);
      if (sample(at.highest) < n) hi = std::max(hi, w[sample(at.highest)] + 1);
    }
    int calls = 0;
    auto below = [&](uint64_t v) { ++calls; return (int)std::count_if(all.begin(), all.end(), [&](uint64_t s) { return s < v; }); };
    const uint64_t v = cut_value(lo, hi, want, below);
    worst = std::max(worst, calls);
    if (below(v) != want) return std::printf("%d samples below the cut for %d\n", below(v), want), 1;
    const size_t words = std::count_if(w.begin(), w.end(), [&](uint64_t x) { return x < v; });
    if (words - words_before > (size_t)(samples * kCutStride + kCutRuns * (kCutStride - 1))) return std::printf("a part of %zu\n", words - words_before), 1;
    words_before = words;
  }
  std::printf("%d\n", worst);
  return n - words_before > (size_t)(samples * kCutStride + kCutRuns * (kCutStride - 1));
}
"""


@pytest.fixture(scope="module")
def cuts(tmp_path_factory):
    d = tmp_path_factory.mktemp("cuts")
    (d / "c.cpp").write_text(CUTS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", build.CSRC, str(d / "c.cpp"), "-o", str(d / "c")], check=True)
    return str(d / "c")


@pytest.mark.parametrize("kind", range(8))
@pytest.mark.parametrize("samples", [32, 48])
def test_merge_cuts_have_the_samples_asked_for_below_them(cuts, samples, kind):
    # a last run of no, one, hardly any, half and almost all its words, behind two to thirty-one whole ones
    for n in [2049, 2112, 2648, 2688, 3071, 3072, 3073, 4600, 8193, 8300, 16384, 20000, 22331, 31745, 32767, 32768]:
        r = subprocess.run([cuts, str(n), str(samples), str(kind)], capture_output=True, text=True)
        assert r.returncode == 0, (n, r.stdout)
        assert int(r.stdout) <= 2 + 57, n                # two ends and the bits of key and index below a common segment
