// When the 128-query attention shape reads the rows of K and V itself (attn_rows_kernel) instead of tiles laid out before it.  Plain C++
// without the device: checked on the host.
#pragma once
#include <cstddef>
#include <cstdint>

namespace basa {

// Is that the faster way?  Its loop is 9 % slower for it (addresses, twice the reads of V^T, and the loads of the next tile are waited for
// in mid-tile); laying out the tiles takes a launch and four times kv_bytes (of one of the two).  attention_us: plan_call's estimate for
// the shape and the splits that it chose.  Attention call, tiles -> rows: 256 queries of 32768, keep 25 %, 32 heads on 8: 73.3 -> 56.7 us,
// 32 on 32: 108 -> 59.5; 32 of 100000, keep 10 %: 67 -> 44; 8 heads, L = 4000, keep 10 %: 22.1 -> 16.8, L = 2472, keep 50 %: 35.2 -> 32.1, L =
// 8000: 145.5 -> 141.5; 2 heads, L = 600, d = 64: 14.6 -> 11.5; 32 heads, 1024 queries of 100000, keep 5 %, of which the bitmaps would
// lay out a third: 173 -> 109; long calls of short lists: 2 heads, L = 100000, keep 5 %: 567 -> 563; kept at tiles: 8 heads on 2, L = 8000:
// 137.9 / 140.0; 32 on 8, L = 4000: 124.4 / 125.0.
// At d = 64 a whole list with a compute unit to itself has nothing to hide the longer loop behind, 0.14 us in each tile of 0.8.  Tiles /
// rows, keep 75 %, B = 64: 8 heads on 2, L = 1200: 18.8 / 19.4, 3145: 38.1 / 41.8; 1 head, 2472: 30.6 / 33.3; 8 heads, 2472: 33.0 / 34.2; rows: 8
// heads, 1200: 19.6 / 19.5, keep 50 %, B = 128: 14.4 / 13.8.  Both lines over 550 calls of 60 to 260 thousand rows: 0.08 % slower than the
// better of the two on average, 5 % at most.
inline bool rows_pay(size_t kv_bytes, double attention_us, bool d64_alone) {
  const double tiles_us = 4.0 * (double)kv_bytes / 5.6e6;
  return d64_alone ? 3.4 + tiles_us > 0.19 * attention_us : 4.0 + tiles_us > 0.09 * attention_us;
}
// The kernel forms a row's offset from the head's first as a product of two 24-bit numbers, in 32 bits.
inline bool offsets_fit(int64_t L, int64_t stride_l) {
  return stride_l < 1 << 23 && L < 1 << 24 && L * stride_l * 2 < (int64_t)1 << 32;
}

}  // namespace basa
