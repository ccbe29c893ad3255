// Which tiles a norm sort starts from, by its sizes, and where its merge cuts their runs.  Plain C++ without the device: checked on
// the host.
#pragma once
#include <algorithm>
#include <cstdint>

namespace basa {

constexpr int kTile = 4096;          // elements sorted per workgroup in LDS (32 KB); kSmallTile for calls of fewer words
constexpr int kSmallTile = 1024;
constexpr int64_t kMidWords = 1 << 21;

struct SortPlan {
  bool few;                          // runs are ranked against each other over the device instead of merged
  int tile;
};

// One tensor, or two (rows1 > 0) through the same launches: rows of L tokens of `token_bytes` each, sorted in runs of `window`
// tokens if that is not 0.  cached: the tokens are loaded through the caches.
inline SortPlan plan_sort(int64_t rows0, int L0, int64_t rows1, int L1, int window, int token_bytes, bool cached) {
  const int64_t words = rows0 * L0 + rows1 * L1;
  const int longest = rows1 > 0 ? std::max(L0, L1) : L0, run = window > 0 ? std::min(window, longest) : longest;
  // Few words: tiles of 1024 tokens, four times as many workgroups to read the rows, and ranking, which spreads the
  // merges over the device; many words: tiles of 4096 and the merging kernels, which move each word once or
  // twice.  The line, rows x tokens (d = 128, tile pass + merges, small against large tiles): 16 x 8192 31 against 75 us,
  // 64 x 8192 61 / 78, 32 x 16384 69 / 88, 16 x 32768 93 / 102; 64 x 16384 116 / 96, 8 x 100000 196 / 135.
  if (words <= (1 << 19)) {
    if (!cached || run <= kSmallTile || run > 8 * 512) return {true, kSmallTile};
    // Tiles of 512 where eight of them make a run and one ranking pass merges them either way: twice the workgroups read the
    // rows and each sorts half as much, as long as there are no more of them than the compute units take at once.  Sort, tiles of
    // 1024 -> 512, 256 bytes a token, runs of 4096: 16 rows 21.6 -> 16.8 us, 32: 22.0 -> 18.4, kept at 1024: 64: 27.6 / 31.4, 128:
    // 44 / 51; longer where the second tile of 1024 is hardly used (runs of 1500: 20 rows 21.4 -> 16.0, 349: 47.5 -> 47.0) and with
    // 128 bytes a token (runs of 4096, 64 rows: 21.1 / 21.2, kept at 1024: 98: 31.1 / 33.4).
    const bool short_tokens = token_bytes <= 128;
    if (run <= 3 * 512 || (short_tokens && run <= 4 * 512)) return {true, 512};
    auto tiles = [&](int64_t rows, int L) {
      const int w = std::min(run, L);
      return rows * ((L + w - 1) / w) * ((w + 511) / 512);
    };
    const int64_t count = tiles(rows0, L0) + (rows1 > 0 ? tiles(rows1, L1) : 0);
    return {true, count <= (short_tokens ? 640 : run <= 4 * 512 ? 400 : 256) ? 512 : kSmallTile};
  }
  // Up to kMidWords the tiles stay at 1024: 4096-token tiles are one or two workgroups to a compute unit there, whose bitonic networks
  // nothing hides.  Whole sort, d = 128, large tiles / small: 1.0 million words in runs of 1024: 92 / 50 us, 1500: 87 / 72, 2048: 79 / 59,
  // 8300: 114 / 81, 12000: 88 / 73, 16384: 90 / 75, 32768: 104 / 81; 2.0 million: 2048: 128 / 108, 8300: 139 / 136, 16384: 139 / 129, 32768:
  // 154 / 137.  The line is older than the merge cut by samples (sort.hip), which the small tiles have here from runs of 2049 on: beyond it,
  // kept at large tiles, 2.1 million words in runs of 32768: 187 / 148, 2.5: 191 / 174, 3.0: 197 / 202, 4.0: 249 / 260, 16384: 229 / 249, 2.4
  // in runs of 8300: 199 / 165.
  if (words > kMidWords) return {false, kTile};
  if (run <= 2 * kSmallTile || run > 2 * kTile) return {false, kSmallTile};
  // Runs of 2049 to 8192 tokens.  One large tile is the whole run: 3000 tokens, 1.0 and 2.0 million words: 86 / 78 and 127 / 128, 4096: 70 / 70 and
  // 117 / 128.  Or two are, and a merge pass: small tiles for 129 to 256 runs, where the large ones are more than one to a compute unit and
  // the small ones at most five (132 of 5000: 101 / 61, 256: 112 / 86, 132 of 8192: 112 / 82, 160: 114 / 86).  These lines too are older than the
  // present merge; kept at large tiles: 128 of 5000: 74 / 59, 260: 144 / 101, 128 of 8192: 81 / 73, 162: 114 / 93, 200 of 7000: 115 / 104.
  if (run <= kTile) return {false, kTile};
  const int64_t runs = rows0 * ((L0 + run - 1) / run) + (rows1 > 0 ? rows1 * ((L1 + run - 1) / run) : 0);
  return {false, runs > 128 && runs <= 256 && words <= 5 * 256 * kSmallTile ? kSmallTile : kTile};
}

// The merge that is cut by samples (sort.hip): up to kCutRuns neighbouring runs of kSmallTile words, every kCutStride-th word of a
// run a sample.
constexpr int kCutRuns = 32, kCutStride = kSmallTile / 16;
// A value with exactly `want` of the samples of `words` words below it lies between two that are known by their numbers in the runs.
// Sample `lowest`: the smallest of the runs' has at most `want` below it.  Sample `highest`: behind the largest there are at least
// `want`, those of the whole runs alone (the last run may be short and lack it).  For want > 0, a multiple of 16, kCutStride * want <
// words: then there are two runs or more, and `highest` is at most 15.  (With sample `lowest` at both ends, a short last run that lacks
// it left the upper end one value short, or at the largest of all values: 40 steps of 0.2 us in place of 6.  Whole sort,
// 196 rows of 5354: 89.3 -> 81.9 us, 26 of 30222: 83.6 -> 77.9.)
struct CutBracket { int lowest, highest; };
constexpr CutBracket cut_bracket(int want, int words) {
  return {want / ((words + kSmallTile - 1) / kSmallTile), (want - 1) / (words / kSmallTile)};
}
// That value: below(lo) <= want <= below(hi), and below() grows by at most one with each step of its argument, the words being distinct.
template <class Below>
constexpr uint64_t cut_value(uint64_t lo, uint64_t hi, int want, Below&& below) {
  if (below(lo) == want) return lo;        // mostly: the runs are much alike
  if (below(hi) == want) return hi;        // (no value between the two need have it)
  while (hi - lo > 1) {                    // below(lo) < want < below(hi)
    const uint64_t v = lo + ((hi - lo) >> 1);
    const int c = below(v);
    if (c == want) return v;
    if (c > want) hi = v; else lo = v;
  }
  return lo;                               // (cannot be)
}

}  // namespace basa
