// Norm ranking (Sec. 3.3, Eq. 9-10; Alg. 1 steps 1-2): sort keys and a segmented
// merge sort of (key, index) pairs, one segment per (head, window).
//
// Key of a token = fp32 rounding of the fp64 sum of squares of its d values.  Each
// pair is packed into one 64-bit word, [segment : 6][key bits without the sign : 31][token
// index : 27]: keys are non-negative floats, whose bit patterns order like the values, so an
// unsigned compare of the packed words orders by segment, then key, and breaks ties by lower
// index, which also makes every word distinct (no stability concerns in the sort).  The
// segment field is 0 unless the caller gave a list of segments of unequal length; those are
// sorted as ONE sequence per head, and the segment field keeps every segment in its range.
#include <algorithm>
#include <type_traits>
#include "common.hpp"
#include "sort_plan.hpp"

namespace basa {
namespace {

constexpr int kSortThreads = 256;
constexpr int kMergeItems = 8;       // outputs per thread in a merge pass
constexpr int kMergeChunk = kSortThreads * kMergeItems;   // 2048 outputs per workgroup
constexpr int kIdxBits = 27;
static_assert((1 << kIdxBits) == kMaxSortLen && BASA_MAX_SEGMENTS < 64, "fields of the packed word");
__device__ __forceinline__ uint64_t pack_word(int seg, float key, int idx) {
  return ((uint64_t)(uint32_t)seg << 58) | ((uint64_t)(__float_as_uint(key) & 0x7fffffffu) << kIdxBits) | (uint32_t)idx;
}
__device__ __forceinline__ int32_t idx_of_word(uint64_t w) { return (int32_t)((uint32_t)w & ((1u << kIdxBits) - 1u)); }

// ---------------------------------------------------------------------------------
// Keys + tile sort in one kernel.  A workgroup owns one tile of up to kTile consecutive tokens
// of a segment: it streams their rows (a row of d elements is 16-byte chunks spread over LPR
// adjacent lanes; two batches of 8 rows per thread in flight), writes the packed (key, index)
// words into LDS, sorts them there with a bitonic network, and writes the sorted tile (or,
// when the tile is the whole segment, the permutation itself).  Workgroups of a compute unit
// are in different phases, so the LDS-bound sort of one hides under the HBM-bound key pass of
// the others.
// Segment s of a head covers [s*W, min((s+1)*W, L)); tiles never straddle segments.
// Up to two tensors of the same d and dtype are handled by one launch: rows blockIdx.y < BH0 belong
// to x0 (geometry g0), the rest to x1 (g1); packed words of x1 follow those of x0.
// ---------------------------------------------------------------------------------
struct SegGeom {
  int L, W, segs, tiles_per_seg;
};

// ---- the tile's bitonic network, 16 words per thread in registers ------------------------
// Word i of the tile lives at LDS slot i + i/16 (one pad word per 16: a thread's 16 consecutive
// words, and the other two ownership patterns below, then hit distinct banks).
__device__ __forceinline__ int tile_slot(int i) { return i + (i >> 4); }

// Three ways of dealing the 4096 = 2^12 words to 256 threads x 16 registers; in layout G the
// register number is index bits 4G+3 .. 4G, so the compare-exchange stages whose distance 2^b
// has b in that range work on registers only.
template <int G>
__device__ __forceinline__ int word_of(int t, int r) {
  if (G == 0) return (t << 4) | r;
  if (G == 1) return ((t >> 4) << 8) | (r << 4) | (t & 15);
  return (r << 8) | t;
}
template <int G>
__device__ __forceinline__ void regs_from_lds(uint64_t (&v)[16], const uint64_t* buf, int t) {
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = buf[tile_slot(word_of<G>(t, r))];
}
template <int G>
__device__ __forceinline__ void regs_to_lds(const uint64_t (&v)[16], uint64_t* buf, int t) {
#pragma unroll
  for (int r = 0; r < 16; ++r) buf[tile_slot(word_of<G>(t, r))] = v[r];
}
// Stages of the merge step with block size k whose compare distance 2^b has b_lo <= b <= b_hi,
// all inside layout G's register bits.  A pair is ordered ascending where index bit log2(k) is 0.
template <int G>
__device__ __forceinline__ void stages_in_regs(uint64_t (&v)[16], int t, int k, int b_hi, int b_lo) {
  asm volatile("" : "+v"(t));      // as in relayout(): recompute the word indices here
#pragma unroll
  for (int lb = 3; lb >= 0; --lb) {
    const int b = 4 * G + lb;
    if (b <= b_hi && b >= b_lo) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (r & (1 << lb)) continue;
        const int r2 = r | (1 << lb);
        const bool up = (word_of<G>(t, r) & k) == 0;
        const uint64_t a = v[r], c = v[r2];
        const bool swap = (a > c) == up;
        v[r] = swap ? c : a;
        v[r2] = swap ? a : c;
      }
    }
  }
}
// Moves the tile from layout A (registers) to layout B (registers) through LDS.
template <int A, int B>
__device__ __forceinline__ void relayout(uint64_t (&v)[16], uint64_t* buf, int t) {
  // the slot addresses are recomputed at every use (two integer ops each): left to itself the
  // compiler keeps all 48 of them in registers across the whole network and halves the occupancy
  asm volatile("" : "+v"(t));
  regs_to_lds<A>(v, buf, t);
  __syncthreads();
  regs_from_lds<B>(v, buf, t);
  __syncthreads();                 // everyone has read before anyone writes the next layout
}
// Sorts the kTile words in buf (slots tile_slot(i)) ascending; ends with the words back in buf.
__device__ __forceinline__ void sort_tile_in_lds(uint64_t* buf, int t) {
  static_assert(kTile == 4096 && kSortThreads == 256, "16 words per thread, 12 index bits in three groups of 4");
  uint64_t v[16];
  regs_from_lds<0>(v, buf, t);
  __syncthreads();
  for (int m = 1; m <= 12; ++m) {
    const int k = 1 << m;          // k = 4096: bit 12 of an index is always 0, everything ascending
    if (m > 8) {
      relayout<0, 2>(v, buf, t);
      stages_in_regs<2>(v, t, k, m - 1, 8);
      relayout<2, 1>(v, buf, t);
      stages_in_regs<1>(v, t, k, 7, 4);
      relayout<1, 0>(v, buf, t);
      stages_in_regs<0>(v, t, k, 3, 0);
    } else if (m > 4) {
      relayout<0, 1>(v, buf, t);
      stages_in_regs<1>(v, t, k, m - 1, 4);
      relayout<1, 0>(v, buf, t);
      stages_in_regs<0>(v, t, k, 3, 0);
    } else {
      stages_in_regs<0>(v, t, k, m - 1, 0);
    }
  }
  regs_to_lds<0>(v, buf, t);
  __syncthreads();
}

// ---- the network of a small tile: 1024 or 512 words, 256 or 512 threads, W = 4, 2 or 1 words per thread ----
// Wave w sorts words 64 W w .. 64 W (w + 1) - 1 by itself (index = W lane + register: the low index bits in registers, six
// exchanged between lanes, no barrier); the runs of the waves are then ranked against each other in LDS.  Returns in
// rank[r] the place of v[r] in the tile (padding words, all alike, get places past the last real word).
template <int W>
__device__ __forceinline__ void sort_in_wave(uint64_t (&v)[W], int lane) {
  constexpr int kRegBits = W == 4 ? 2 : W == 2 ? 1 : 0;
#pragma unroll
  for (int m = 1; m <= 6 + kRegBits; ++m) {
    const int k = 1 << m;              // in the last step beyond the indices of a wave, everything ascending
#pragma unroll
    for (int b = m - 1; b >= 0; --b) {
      if (b < kRegBits) {
#pragma unroll
        for (int r = 0; r < W; ++r) {
          if (r & (1 << b)) continue;
          const int r2 = r | (1 << b);
          const bool up = ((W * lane + r) & k) == 0;
          const uint64_t a = v[r], c = v[r2];
          const bool swap = (a > c) == up;
          v[r] = swap ? c : a;
          v[r2] = swap ? a : c;
        }
      } else {
        const bool up = ((W * lane) & k) == 0, lower = (lane & (1 << (b - kRegBits))) == 0;
#pragma unroll
        for (int r = 0; r < W; ++r) {
          const uint64_t o = __shfl_xor((unsigned long long)v[r], 1 << (b - kRegBits));
          const bool take = (o < v[r]) == (lower == up);
          v[r] = take ? o : v[r];
        }
      }
    }
  }
}
template <int W, int kWaves>
__device__ __forceinline__ void rank_small_tile(uint64_t (&v)[W], int (&rank)[W], uint64_t* buf, int t) {
  constexpr int kRun = 64 * W, kOthers = kWaves - 1;
  const int lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int r = 0; r < W; ++r) v[r] = buf[tile_slot(W * t + r)];
  sort_in_wave<W>(v, lane);
#pragma unroll
  for (int r = 0; r < W; ++r) {
    buf[tile_slot(W * t + r)] = v[r];          // (each wave rewrites the words it read)
    rank[r] = W * lane + r;
  }
  __syncthreads();
  // Words below v[r] in the runs of the other waves: a binary search in each, side by side.  A position P in a run is kept as
  // its slot P + P/16, which a step moves by a constant: every probe is one LDS read at an immediate offset, one
  // compare and one conditional add.
  int pos[kOthers][W];
#pragma unroll
  for (int j = 0; j < kOthers; ++j)
#pragma unroll
    for (int r = 0; r < W; ++r) pos[j][r] = tile_slot(((wave + 1 + j) & kOthers) * kRun);
  auto probe = [&](auto step, auto move) {       // is word P + step - 1 below v[r]?  Then P moves on by `step`
    constexpr int kStep = decltype(step)::value, kMove = decltype(move)::value;
    constexpr int kOff = kStep >= 16 ? kMove - 2 : kStep - 1;
    uint64_t w[kOthers][W];
#pragma unroll
    for (int j = 0; j < kOthers; ++j)
#pragma unroll
      for (int r = 0; r < W; ++r) w[j][r] = buf[pos[j][r] + kOff];
#pragma unroll
    for (int j = 0; j < kOthers; ++j)
#pragma unroll
      for (int r = 0; r < W; ++r) pos[j][r] = w[j][r] < v[r] ? pos[j][r] + kMove : pos[j][r];
  };
#define BASA_PROBE(S) probe(std::integral_constant<int, S>{}, std::integral_constant<int, S >= 16 ? S + S / 16 : S>{})
  if constexpr (W == 4) BASA_PROBE(128);
  if constexpr (W >= 2) BASA_PROBE(64);
  BASA_PROBE(32); BASA_PROBE(16); BASA_PROBE(8); BASA_PROBE(4); BASA_PROBE(2); BASA_PROBE(1);
#undef BASA_PROBE
  // P <= kRun - 1 now; word P itself decides between P and P + 1
#pragma unroll
  for (int j = 0; j < kOthers; ++j) {
    const int run0 = tile_slot(((wave + 1 + j) & kOthers) * kRun);
#pragma unroll
    for (int r = 0; r < W; ++r) {
      const int slot = pos[j][r] - run0;         // P + P/16
      rank[r] += slot - slot / 17 + (buf[pos[j][r]] < v[r] ? 1 : 0);
    }
  }
}

template <bool kBf16, int kD, int kTileT, bool kStream, int kThreads = kSortThreads>
__device__ __forceinline__ void norm_tile_sort(int bx, int by, const TensorView& x0, const TensorView& x1, int BH0,
                                               uint64_t* __restrict__ out, int32_t* __restrict__ perm0,
                                               int32_t* __restrict__ perm1, float* __restrict__ keys_out, const SegGeom& g0,
                                               const SegGeom& g1, const SegList& sl) {
  constexpr int kElem = kBf16 ? 2 : 4;
  constexpr int LPR = kD * kElem / 16;          // lanes per row: 8, 16 or 32
  constexpr int kRowsPerIter = kThreads / LPR;
  constexpr int kIters = 8;
  constexpr int kRowsPerPass = kRowsPerIter * kIters;
  static_assert(kTileT % kRowsPerPass == 0, "a tile is a whole number of passes");
  __shared__ uint64_t buf[kTileT + kTileT / 16];

  const bool second = by >= BH0;
  const SegGeom& g = second ? g1 : g0;
  const int bh = second ? by - BH0 : by;
  const int seg = bx / g.tiles_per_seg;
  const int tile = bx - seg * g.tiles_per_seg;
  const int seg_end = min((seg + 1) * g.W, g.L);
  const int start = seg * g.W + tile * kTileT;
  if (start >= seg_end) return;
  const int n = min(kTileT, seg_end - start);
  const int64_t hb = (int64_t)bh * g.L;
  const TensorView& x = second ? x1 : x0;
  if (second) out += (int64_t)BH0 * g0.L;
  int32_t* perm_out = second ? perm1 : perm0;
  const char* base = reinterpret_cast<const char*>(x.ptr) + x.head_offset(bh) * kElem;
  const int sub = threadIdx.x % LPR;
  const int rig = threadIdx.x / LPR;
  // segment of the tile's first token; nearly every tile lies inside one segment
  int seg_lo = 0;
  for (int j = 1; j < sl.n; ++j) seg_lo += (start >= sl.bound[j]) ? 1 : 0;
  const bool one_segment = sl.n <= 1 || start + n <= sl.bound[seg_lo + 1];

  // ---- phase 1: keys of tokens start .. start+n-1 into buf
  // Every load is unconditional, its row clamped into the tile (a row past the end reads the
  // tile's last row, whose key is never written): loads inside branches make the compiler wait
  // for ALL outstanding loads at the join, the prefetch of the next pass included, and the double
  // buffering is lost.
  const int passes = (n + kRowsPerPass - 1) / kRowsPerPass;
  auto load_pass = [&](int pass, uint4 (&raw)[kIters]) {
    // A pass past the last (the loop below asks for up to four of them) has every lane read the tile's
    // first 16 bytes, one cache line per instruction, instead of the last pass again: the loads are
    // streaming loads, which nothing caches, so a repeated pass would cost its 32 KB of HBM traffic
    // again (an eighth of the tile in all).
    const bool live = pass < passes;             // uniform over the workgroup
    const int sub_l = live ? sub : 0;
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      const int loc = live ? min(pass * kRowsPerPass + it * kRowsPerIter + rig, n - 1) : 0;
      // (streaming loads in large calls: the pass takes 0.416 instead of 0.431 ms at 128K, the rows no longer push
      //  the sort words being written out of the cache.  Bit-cast into uint4, not held as the builtin's vector type: the compiler
      //  rotates such vectors through the three buffers as whole registers, copies that count as uses of loads still in
      //  flight.  And written here: as a function of row and chunk it makes another schedule of the whole kernel, 60.4 us
      //  instead of 57.0 for 200 x 3000, d = 128, fp32 64 x 880: 18.9 and 17.6.)
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      const u32x4* src = reinterpret_cast<const u32x4*>(base + (int64_t)(start + loc) * x.stride_l * kElem) + sub_l;
      raw[it] = __builtin_bit_cast(uint4, kStream ? __builtin_nontemporal_load(src) : *src);
    }
  };
  auto keys_of_pass = [&](int pass, const uint4 (&cur)[kIters]) {
    // per-lane partial sums of the kIters rows this lane contributes to
    double acc[kIters];
#pragma unroll
    for (int it = 0; it < kIters; ++it) {
      acc[it] = 0.0;
      const uint32_t w[4] = {cur[it].x, cur[it].y, cur[it].z, cur[it].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (kBf16) {
          // |x| as a double, built from the 15 exponent+mantissa bits of the bf16 (the float to
          // double conversion instruction is many times slower than these two integer ops): the
          // high word of the double is bits << 13 plus the exponent rebias (1023-127) << 20, the
          // low word is zero.  A zero or subnormal bf16 (exponent field 0) comes out as a value
          // below 2^-126 instead; its square, below 2^-252, is lost against any sum that can
          // round to a non-zero fp32 key (>= 2^-150), exactly as the true square would be.
          const double lo = __hiloint2double((int)((__builtin_amdgcn_ubfe(w[i], 0, 15) << 13) + 0x38000000u), 0);
          const double hi = __hiloint2double((int)((__builtin_amdgcn_ubfe(w[i], 16, 15) << 13) + 0x38000000u), 0);
          acc[it] = fma(lo, lo, acc[it]);
          acc[it] = fma(hi, hi, acc[it]);
        } else {
          const double v = (double)__uint_as_float(w[i]);
          acc[it] = fma(v, v, acc[it]);
        }
      }
    }
    // Reduction over the LPR lanes of a row, all kIters rows at once: in the step with lane
    // distance 2^b a lane hands the half of its partial sums that its partner keeps to the
    // partner and halves its own set (8 -> 4 -> 2 -> 1 sums in 7 exchanges instead of 24), so
    // that after three steps lane `sub` holds one row, iteration 4*bit0 + 2*bit1 + bit2 of sub.
    static_assert(kIters == 8 && LPR >= 8, "the exchange pattern below is written for 8 rows");
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const bool upper = (sub >> b) & 1;
      const int m = kIters >> (b + 1);
#pragma unroll
      for (int i = 0; i < m; ++i) {
        const double give = upper ? acc[i] : acc[i + m];
        const double keep = upper ? acc[i + m] : acc[i];
        acc[i] = keep + __shfl_xor(give, 1 << b, LPR);
      }
    }
#pragma unroll
    for (int off = 8; off < LPR; off <<= 1) acc[0] += __shfl_xor(acc[0], off, LPR);
    const int it_mine = 4 * (sub & 1) + (sub & 2) + ((sub >> 2) & 1);
    const int loc = pass * kRowsPerPass + it_mine * kRowsPerIter + rig;
    if (sub < 8 && loc < n) {
      const float key = (float)acc[0];
      // (the segment of the tile's first token; a tile that straddles a boundary is put right below,
      //  outside this loop, whose loads the compiler can then count exactly)
      buf[tile_slot(loc)] = pack_word(seg_lo, key, start + loc);
      if (keys_out) keys_out[hb + start + loc] = key;
    }
  };
  // three batches of rows: two are in flight while the third is turned into keys (a pass past the last
  // writes nothing: its positions lie beyond n)
  uint4 b0[kIters], b1[kIters], b2[kIters];
  load_pass(0, b0);
  load_pass(1, b1);
  load_pass(2, b2);
  for (int pass = 0; pass < passes; pass += 3) {
    keys_of_pass(pass, b0);
    load_pass(pass + 3, b0);
    keys_of_pass(pass + 1, b1);
    load_pass(pass + 4, b1);
    keys_of_pass(pass + 2, b2);
    load_pass(pass + 5, b2);
  }
  if (!one_segment) {              // workgroup-uniform and rare: some tokens belong to later segments
    // (the keys stored in the loop above have to be in LDS before the barrier; the compiler's own wait
    //  was found missing on this path by lds_wait_audit, so it is spelt out)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kThreads) {
      int sg = seg_lo;
      for (int j = seg_lo + 1; j < sl.n; ++j) sg += (start + i >= sl.bound[j]) ? 1 : 0;
      if (sg != seg_lo) {
        const uint64_t w = buf[tile_slot(i)];
        buf[tile_slot(i)] = (w & ((1ull << 58) - 1ull)) | ((uint64_t)(uint32_t)sg << 58);
      }
    }
  }
  for (int i = n + threadIdx.x; i < kTileT; i += kThreads) buf[tile_slot(i)] = ~0ull;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();

  // ---- phase 2: the words of the tile into order
  if constexpr (kTileT <= kSmallTile) {
    constexpr int W = kTileT / kThreads;
    uint64_t v[W];
    int rank[W];
    rank_small_tile<W, kThreads / 64>(v, rank, buf, threadIdx.x);
#pragma unroll
    for (int r = 0; r < W; ++r) {
      if (v[r] == ~0ull) continue;             // padding
      if (perm_out) perm_out[hb + start + rank[r]] = idx_of_word(v[r]);
      else out[hb + start + rank[r]] = v[r];
    }
    return;
  }
  sort_tile_in_lds(buf, threadIdx.x);
  if (perm_out) {
    for (int i = threadIdx.x; i < n; i += kThreads) perm_out[hb + start + i] = idx_of_word(buf[tile_slot(i)]);
  } else {
    // (streaming stores, like the loads of the rows: another 3 % of this kernel)
    for (int i = threadIdx.x; i < n; i += kThreads) __builtin_nontemporal_store(buf[tile_slot(i)], &out[hb + start + i]);
  }
}

template <bool kBf16, int kD, int kTileT, int kThreads, bool kStream>
__global__ __launch_bounds__(kThreads) void norm_tile_sort_kernel(TensorView x0, TensorView x1, int BH0,
                                                                      uint64_t* __restrict__ out,
                                                                      int32_t* __restrict__ perm0,
                                                                      int32_t* __restrict__ perm1,
                                                                      float* __restrict__ keys_out, SegGeom g0,
                                                                      SegGeom g1, SegList sl, int tiles1) {
  int bx = blockIdx.x, by = blockIdx.y;
  if (tiles1 > 0) {                            // sequences of different lengths: one row of workgroups, those of x1 first
    const bool second = bx < tiles1;
    const int i = second ? bx : bx - tiles1, per_row = second ? g1.segs * g1.tiles_per_seg : g0.segs * g0.tiles_per_seg;
    by = i / per_row;
    bx = i - by * per_row;
    by += second ? BH0 : 0;
  }
  norm_tile_sort<kBf16, kD, kTileT, kStream, kThreads>(bx, by, x0, x1, BH0, out, perm0, perm1, keys_out, g0, g1, sl);
}
template <int kD>
struct SmallSortJob {
  TensorView q, k;
  uint64_t* out;
  int32_t *perm_q, *perm_k;                // null: more than one tile
  SegGeom g;
  __device__ __forceinline__ void run(int block) const {
    SegList whole;
    whole.n = 0;
    const int by = block / g.tiles_per_seg;
    norm_tile_sort<true, kD, kSmallTile, false>(block - by * g.tiles_per_seg, by, q, k, q.heads, out, perm_q, perm_k, nullptr, g, g, whole);
  }
};

// ---------------------------------------------------------------------------------
// Merge pass: sorted runs of `run` elements are merged pairwise inside each segment.
// One workgroup produces kMergeChunk consecutive outputs of one pair, located with a
// merge-path search on the pair's two runs.
// ---------------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ int merge_path(const T* A, int na, const T* Bv, int nb, int diag) {
  int lo = max(0, diag - nb), hi = min(diag, na);
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (A[mid] < Bv[diag - 1 - mid]) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// The same on LDS, word i at slot i + i / kPer: the threads of a wave start kPer outputs apart, and without the pad their
// reads and writes meet in a few banks (4 x 10^6 words: 18.4 -> 16.9 us a pass).
template <int kPer>
__host__ __device__ constexpr __forceinline__ int padded(int i) { return i + i / kPer; }
template <int kPer, class T>
__device__ __forceinline__ int merge_path_lds(const T* buf, int a0, int na, int b0, int nb, int diag) {
  int lo = max(0, diag - nb), hi = min(diag, na);
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (buf[padded<kPer>(a0 + mid)] < buf[padded<kPer>(b0 + diag - 1 - mid)]) lo = mid + 1; else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(kSortThreads) void merge_pass_kernel(const uint64_t* __restrict__ in,
                                                                  uint64_t* __restrict__ out,
                                                                  int32_t* __restrict__ perm0,
                                                                  int32_t* __restrict__ perm1, int BH0,
                                                                  SegGeom g, int run,
                                                                  int chunks_per_pair, int pairs_per_seg) {
  constexpr int kPer = kMergeItems;
  __shared__ uint64_t buf[kMergeChunk + kMergeChunk / kPer];
  __shared__ int split[2];
  const int bh = blockIdx.y;
  int id = blockIdx.x;
  const int chunk = id % chunks_per_pair; id /= chunks_per_pair;
  const int pair = id % pairs_per_seg;
  const int seg = id / pairs_per_seg;
  const int seg_end = min((seg + 1) * g.W, g.L);
  const int a0 = seg * g.W + pair * 2 * run;
  if (a0 >= seg_end) return;
  const int na = min(run, seg_end - a0);
  const int b0 = a0 + na;
  const int nb = min(run, seg_end - b0);
  const int total = na + nb;
  const int diag0 = chunk * kMergeChunk;
  if (diag0 >= total) return;
  const int diag1 = min(diag0 + kMergeChunk, total);
  const int64_t hb = (int64_t)bh * g.L;
  int32_t* perm_out = bh < BH0 ? perm0 : (perm1 ? perm1 - (int64_t)BH0 * g.L : nullptr);
  const uint64_t* A = in + hb + a0;
  const uint64_t* Bv = in + hb + b0;

  if (threadIdx.x < 2) split[threadIdx.x] = merge_path(A, na, Bv, nb, threadIdx.x == 0 ? diag0 : diag1);
  __syncthreads();
  const int as = split[0], ae = split[1];
  const int bs = diag0 - as, be = diag1 - ae;
  const int ca = ae - as, cb = be - bs;          // ca + cb == diag1 - diag0
  const int n = ca + cb;
  {
    // the chunk's share of the two runs, side by side in LDS; the kMergeItems loads of a thread
    // are unconditional (index clamped into the chunk, n >= 1) so that they are in flight together
    uint64_t w[kMergeItems];
#pragma unroll
    for (int e = 0; e < kMergeItems; ++e) {
      const int i = min(e * kSortThreads + (int)threadIdx.x, n - 1);
      w[e] = i < ca ? A[as + i] : Bv[bs + i - ca];
    }
#pragma unroll
    for (int e = 0; e < kMergeItems; ++e) {
      const int i = e * kSortThreads + threadIdx.x;
      if (i < n) buf[padded<kPer>(i)] = w[e];
    }
  }
  __syncthreads();

  const int d0 = min(threadIdx.x * kMergeItems, n);
  const int d1 = min(d0 + kMergeItems, n);
  int ia = merge_path_lds<kPer>(buf, 0, ca, ca, cb, d0);
  int ib = d0 - ia;
  // merge kMergeItems outputs into registers, then hand them back through LDS so that the
  // global stores of the workgroup are consecutive
  uint64_t res[kMergeItems];
#pragma unroll
  for (int e = 0; e < kMergeItems; ++e) {
    uint64_t va = ia < ca ? buf[padded<kPer>(ia)] : ~0ull;
    uint64_t vb = ib < cb ? buf[padded<kPer>(ca + ib)] : ~0ull;
    if (va < vb) { res[e] = va; ++ia; } else { res[e] = vb; ++ib; }
  }
  __syncthreads();                       // everyone is done reading the two runs
#pragma unroll
  for (int e = 0; e < kMergeItems; ++e)
    if (d0 + e < d1) buf[padded<kPer>(d0 + e)] = res[e];
  __syncthreads();
  const int64_t obase = hb + a0 + diag0;
  if (perm_out) {
    for (int i = threadIdx.x; i < n; i += kSortThreads) perm_out[obase + i] = idx_of_word(buf[padded<kPer>(i)]);
  } else {
    for (int i = threadIdx.x; i < n; i += kSortThreads) out[obase + i] = buf[padded<kPer>(i)];
  }
}

// ---------------------------------------------------------------------------------
// The first two merge passes in one: 16384 words (128 KB), four neighbouring sorted tiles of 4096, are brought
// into LDS, merged pairwise until they are one run, and written out once, so the words cross the memory system
// one time less.  1024 threads, 16 words each: a thread finds the start
// of its 16 consecutive outputs with a merge-path search in LDS, merges them into registers, and
// the workgroup puts the registers back into LDS between the two levels.  Slots past the end of
// the segment hold the all-ones word, which sorts last (no packed word has segment field 63).
// ---------------------------------------------------------------------------------
constexpr int kQuadThreads = 1024, kQuadItems = 16, kQuadWords = 4 * kTile;
static_assert(kQuadThreads * kQuadItems == kQuadWords, "one word per thread and item");

__global__ __launch_bounds__(kQuadThreads) void merge_quads_kernel(const uint64_t* __restrict__ in,
                                                                   uint64_t* __restrict__ out,
                                                                   int32_t* __restrict__ perm0,
                                                                   int32_t* __restrict__ perm1, int BH0, SegGeom g,
                                                                   int quads_per_seg, int quads_total) {
  extern __shared__ __attribute__((aligned(16))) uint64_t quad[];       // kQuadWords
  const int t = threadIdx.x;
  // A workgroup takes quads blockIdx.x, blockIdx.x + gridDim.x, ... (one or two of them as launched): the words
  // of the next one are requested into registers before this one is merged, so the memory system is
  // not idle while the workgroup works in LDS.
  struct Where { const uint64_t* src; int64_t obase; int n; int32_t* perm_out; };
  auto locate = [&](int id) -> Where {
    const int per_bh = g.segs * quads_per_seg;
    const int bh = id / per_bh, r = id - bh * per_bh;
    const int seg = r / quads_per_seg, q = r - seg * quads_per_seg;
    const int seg_end = min((seg + 1) * g.W, g.L);
    const int a0 = seg * g.W + q * kQuadWords;
    const int64_t hb = (int64_t)bh * g.L;
    Where w;
    w.n = max(0, min(kQuadWords, seg_end - a0));       // 0: the segment ends before this quad
    w.src = in + hb + a0;
    w.obase = hb + a0;
    w.perm_out = bh < BH0 ? perm0 : (perm1 ? perm1 - (int64_t)BH0 * g.L : nullptr);
    return w;
  };
  auto request = [&](const Where& w, uint64_t (&v)[kQuadItems]) {
    // all sixteen loads of a thread in flight together: index clamped, padding applied at the store to LDS
    if (w.n == 0) return;                        // workgroup-uniform: nothing of this quad exists
#pragma unroll
    for (int e = 0; e < kQuadItems; ++e) v[e] = w.src[min(e * kQuadThreads + t, w.n - 1)];
  };
  int id = blockIdx.x;
  if (id >= quads_total) return;
  Where cur = locate(id);
  uint64_t v[kQuadItems];
  request(cur, v);
  for (;;) {
    const int n = cur.n;
#pragma unroll
    for (int e = 0; e < kQuadItems; ++e) quad[e * kQuadThreads + t] = e * kQuadThreads + t < n ? v[e] : ~0ull;
    const int id_next = id + (int)gridDim.x;
    Where nxt = cur;
    if (id_next < quads_total) {               // workgroup-uniform
      nxt = locate(id_next);
      request(nxt, v);
    }
    __syncthreads();
    const int d0 = t * kQuadItems;               // this thread's outputs d0 .. d0 + 15 at every level
#pragma unroll
    for (int run = kTile; run <= 2 * kTile; run *= 2) {
      const int pb = d0 & ~(2 * run - 1);        // first word of the pair of runs these outputs belong to
      const uint64_t* A = quad + pb;
      const uint64_t* Bv = quad + pb + run;
      int ia = merge_path(A, run, Bv, run, d0 - pb);
      int ib = d0 - pb - ia;
      uint64_t res[kQuadItems];
#pragma unroll
      for (int e = 0; e < kQuadItems; ++e) {
        const uint64_t va = ia < run ? A[ia] : ~0ull;
        const uint64_t vb = ib < run ? Bv[ib] : ~0ull;
        if (va <= vb) { res[e] = va; ++ia; } else { res[e] = vb; ++ib; }
      }
      __syncthreads();                           // everyone is done reading the runs
#pragma unroll
      for (int e = 0; e < kQuadItems; ++e) quad[d0 + e] = res[e];
      __syncthreads();
    }
    if (cur.perm_out) {
      for (int i = t; i < n; i += kQuadThreads) cur.perm_out[cur.obase + i] = idx_of_word(quad[i]);
    } else {
      for (int i = t; i < n; i += kQuadThreads) out[cur.obase + i] = quad[i];
    }
    if (id_next >= quads_total) break;
    __syncthreads();                             // the stores above read LDS; the next quad overwrites it
    id = id_next;
    cur = nxt;
  }
}

// ---------------------------------------------------------------------------------
// kG neighbouring runs into one by ranking: the place of a word is its place in its own run plus the number of
// smaller words in each of the others (no two words are equal), found by kG - 1 binary searches side by side.  One
// word per thread, so that a call of few words is spread over the whole device, where merging kernels have a
// workgroup walk thousands of words in LDS; the searches of a wave (neighbouring words) touch the same lines.
// ---------------------------------------------------------------------------------
// Bound by the probes ((kG - 1) log2(run) per word, through L1); 32 rows of 7627 words, 8 runs each: 15.6 us against
// 40 us for the LDS merge of a few workgroups; 2 x 10^6 words in 32 runs: 193 us against 39.
struct RankArgs {
  const uint64_t* in;
  uint64_t* out;
  int32_t *perm0, *perm1;                  // null unless the last pass
  int BH0;
  SegGeom g;
  int run, chunks_per_bh;
};
__device__ __forceinline__ const RankArgs* job_of(const RankArgs& a, int* logical) {
  const int total = gridDim.x;             // a head's words on one XCD: their scattered stores meet in its L2
  *logical = (total & 7) == 0 ? (blockIdx.x & 7) * (total >> 3) + (blockIdx.x >> 3) : blockIdx.x;
  return &a;
}
// Src: the arguments of one problem or of several.  (The body stands in the kernel: as a function that is inlined into one kernel
// for each, the loads of a step came out in three groups instead of two, 8 runs of 6500 words 6.4 -> 7.6 us.)
template <int kG, class Src>
__global__ __launch_bounds__(kSortThreads) void rank_runs_kernel(Src src) {
  int logical;
  const RankArgs* args = job_of(src, &logical);
  if (!args) return;
  const uint64_t* __restrict__ in = args->in;
  uint64_t* __restrict__ out = args->out;
  int32_t* __restrict__ perm0 = args->perm0;
  int32_t* __restrict__ perm1 = args->perm1;
  const SegGeom g = args->g;
  const int BH0 = args->BH0, run = args->run, chunks_per_bh = args->chunks_per_bh;
  const int bh = logical / chunks_per_bh, i = (logical - bh * chunks_per_bh) * kSortThreads + threadIdx.x;
  if (i >= g.L) return;
  const int64_t hb = (int64_t)bh * g.L;
  const int seg = i / g.W, seg0 = seg * g.W, seg_end = min(seg0 + g.W, g.L);
  const int mine = (i - seg0) / run;
  const int base = seg0 + mine / kG * kG * run;          // first word of the group of runs
  const uint64_t v = in[hb + i];
  constexpr int kOthers = kG - 1;
  const int mine_g = mine % kG;
  int start[kOthers], n[kOthers], pos[kOthers];
#pragma unroll
  for (int j = 0; j < kOthers; ++j) {
    start[j] = base + (j < mine_g ? j : j + 1) * run;
    n[j] = max(0, min(run, seg_end - start[j]));
    pos[j] = 0;
  }
  for (int step = run; step > 0; step >>= 1) {           // (run is a power of two)
    uint64_t w[kOthers];
#pragma unroll
    for (int j = 0; j < kOthers; ++j) {
      const int p = min(pos[j] + step, n[j]);
      w[j] = in[hb + (p > 0 ? start[j] + p - 1 : i)];
    }
#pragma unroll
    for (int j = 0; j < kOthers; ++j)
      if (pos[j] + step <= n[j] && w[j] < v) pos[j] += step;
  }
  int rank = (i - seg0) - mine * run;
#pragma unroll
  for (int j = 0; j < kOthers; ++j) rank += pos[j];
  int32_t* perm_out = bh < BH0 ? perm0 : (perm1 ? perm1 - (int64_t)BH0 * g.L : nullptr);
  if (perm_out) perm_out[hb + base + rank] = idx_of_word(v);
  else out[hb + base + rank] = v;
}

// ---------------------------------------------------------------------------------
// Up to 32 neighbouring runs of 1024 words into one, the outputs cut into parts of about `part_samples` x 64 words so that the
// whole device takes part.  Every 64th word of a run is a sample; a part holds the words between two values that have a
// given number of samples below them, which is at most 63 words a run more than asked for.  A workgroup finds its two
// values by bisection (a wave holds all 512 samples, a step is eight compares and as many ballots), counts the words below
// them in each run with one load per run and value, brings its 32 pieces into LDS and merges them pairwise there.
// Bound by the chain of its phases (6 us until the pieces are in LDS, 2.5 us for each of four or five levels of merges), which two or
// three workgroups to a compute unit overlap.  64 rows of 16384: 22 us where a workgroup for every 16384 words, on a quarter of
// the compute units, took 36; 64 rows of 32768: 42 for 50 in two launches.  Dealing the words of a part to bins by value instead of
// merging measured no faster (the keys above a run's last sample fill a few bins), nor did probing three points at a time.
// ---------------------------------------------------------------------------------
constexpr int kCutThreads = 512, kCutLevels = 5;
constexpr int kCutWords = kCutRuns * kSmallTile;          // of a group
constexpr int kPartSamples = 32, kMaxPartSamples = 48;
static_assert(kPartSamples % 16 == 0 && kMaxPartSamples % 16 == 0, "cut_bracket");
constexpr int kCutCap = kMaxPartSamples * kCutStride + kCutRuns * (kCutStride - 1);
constexpr int kCutItems = 8;                              // outputs of a slot; a thread has slots t and (large parts) t + 512
// (a pair of runs leaves part of its last slot unused)
static_assert((2 * kCutThreads - kCutRuns / 2) * kCutItems >= kCutCap, "outputs of the largest part");
// In LDS a word is [0][segment : 6][key : 31][index : 26], which as a double is positive and finite and orders as before: the vector
// unit has a minimum and a maximum of doubles, but none of 64-bit integers (whole sort, with the padding of the slots: 64 rows of 32768 142 -> 138 us, 32: 82.9 -> 80.8, 64 of 16384: 76.8 -> 75.4).
constexpr int kCutIdxBits = kIdxBits - 1;
__device__ __forceinline__ double to_double(uint64_t w) {
  constexpr uint64_t kIdx = (1ull << kCutIdxBits) - 1;
  return __longlong_as_double((long long)((w >> 1 & ~kIdx) | (w & kIdx)));
}
__device__ __forceinline__ int32_t idx_of_double(double x) { return (int32_t)((uint32_t)__double_as_longlong(x) & ((1u << kCutIdxBits) - 1u)); }
__device__ __forceinline__ uint64_t to_word(double x) {
  const uint64_t w = (uint64_t)__double_as_longlong(x);
  return (w >> kCutIdxBits << kIdxBits) | (w & ((1ull << kCutIdxBits) - 1));
}
// (written out: the library's minimum first quiets NaNs, which there are none of, with another instruction for each operand)
__device__ __forceinline__ double min_of(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double max_of(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
struct CutArgs {
  const uint64_t* in;
  uint64_t* out;
  int32_t *perm0, *perm1;                  // null unless the last pass
  int BH0;
  SegGeom g;
  int groups_per_seg, parts, part_samples; // parts: of a whole group
};
__device__ __forceinline__ void cut_merge(const CutArgs& a, int logical) {
  __shared__ double buf[padded<kCutItems>(kCutCap + kCutItems)];      // (a slot reads eight words on, past the last piece too)
  __shared__ int below[2][kCutRuns], start_of[kCutRuns + 1], slot_of[kCutLevels][kCutRuns / 2 + 1];
  __shared__ uint64_t cut[2];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const SegGeom& g = a.g;
  auto at = [](int i) { return padded<kCutItems>(i); };      // (a slot's words in banks of their own)
  int id = logical;
  const int part = id % a.parts; id /= a.parts;
  const int group = id % a.groups_per_seg; id /= a.groups_per_seg;
  const int seg = id % g.segs, bh = id / g.segs;
  const int a0 = seg * g.W + group * kCutWords;
  const int n_group = min(kCutWords, min((seg + 1) * g.W, g.L) - a0);
  const int samples_per_part = a.part_samples, part_words = samples_per_part * kCutStride;
  if (part * part_words >= n_group) return;
  const bool last_part = (part + 1) * part_words >= n_group;
  const uint64_t* __restrict__ in = a.in + (int64_t)bh * g.L + a0;

  // ---- samples: register j of lane l is sample l % 16 of run 4 j + l / 16
  uint64_t s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int pos = (j * 64 + lane) * kCutStride;
    const uint64_t w = in[min(pos, n_group - 1)];
    s[j] = pos < n_group ? w : ~0ull;
  }
  auto samples_below = [&](uint64_t v) {
    int c = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) c += __popcll(__builtin_amdgcn_ballot_w64(s[j] < v));
    return c;
  };
  // ---- waves 0 and 1: the value with part * samples_per_part samples below it, and the one of the next part
  if (wave < 2) {
    const int want = (part + wave) * samples_per_part;
    uint64_t v = wave == 0 ? 0ull : ~0ull;
    if (wave == 0 ? part > 0 : !last_part) {
      const CutBracket at_sample = cut_bracket(want, n_group);
      uint64_t lo = ~0ull, hi = 0ull;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        lo = s[j] < lo ? s[j] : lo;
        hi = s[j] != ~0ull && s[j] > hi ? s[j] : hi;
      }
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        const uint64_t x = __shfl_xor((unsigned long long)lo, off), y = __shfl_xor((unsigned long long)hi, off);
        lo = x < lo ? x : lo;
        hi = y > hi ? y : hi;
      }
      auto of_lane = [&](uint64_t x, int l) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), l) << 32;
      };
      v = cut_value(of_lane(lo, at_sample.lowest), of_lane(hi, at_sample.highest) + 1, want, samples_below);
    }
    if (lane == 0) cut[wave] = v;
  }
  __syncthreads();

  // ---- wave w: the words of runs 4 w .. 4 w + 3 below the two values.  With c samples of a run below, they end among the
  // 63 words behind the last of these.
  {
    uint64_t w[2][4];
    int from[2][4];
    uint64_t mine = s[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) mine = wave == j ? s[j] : mine;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint64_t b = __builtin_amdgcn_ballot_w64(mine < cut[e]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = __popc((uint32_t)(b >> (16 * r)) & 0xffffu);
        from[e][r] = (c - 1) * kCutStride;       // (c = 0: negative, none)
        const int pos = (4 * wave + r) * kSmallTile + max(from[e][r], 0) + lane;
        w[e][r] = in[min(pos, n_group - 1)];
        if (pos >= n_group) w[e][r] = ~0ull;
      }
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = __popcll(__builtin_amdgcn_ballot_w64(w[e][r] < cut[e]));
        if (lane == 0) below[e][4 * wave + r] = from[e][r] < 0 ? 0 : from[e][r] + c;
      }
  }
  __syncthreads();

  // ---- where the pieces go: piece r at start_of[r]; every wave works out the same
  const int lb = lane < kCutRuns ? below[0][lane] : 0, ub = lane < kCutRuns ? below[1][lane] : 0;
  int sum = ub - lb, skip = lb;
#pragma unroll
  for (int off = 1; off < kCutRuns; off <<= 1) {
    const int x = __shfl_up(sum, off);
    if (lane >= off) sum += x;
  }
#pragma unroll
  for (int off = 1; off < kCutRuns; off <<= 1) skip += __shfl_xor(skip, off);
  const int base = __builtin_amdgcn_readfirstlane(skip);
  const int n = __builtin_amdgcn_readlane(sum, kCutRuns - 1);
  const int before = __shfl_up(sum, 1), ends = lane == 0 ? 0 : before;       // lane r: of the pieces before r (32: of all)
  if (wave == 7 && lane <= kCutRuns) start_of[lane] = ends;
  if (wave < kCutLevels) {
    const int pairs = kCutRuns / 2 >> wave, q = min(lane, pairs);
    const int len = __shfl(ends, min(q + 1, pairs) << (wave + 1)) - __shfl(ends, q << (wave + 1));
    int x = (len + kCutItems - 1) / kCutItems;
#pragma unroll
    for (int off = 1; off < kCutRuns / 2; off <<= 1) {
      const int y = __shfl_up(x, off);
      if (lane >= off) x += y;
    }
    if (lane < pairs) slot_of[wave][lane + 1] = x;
    if (lane == 0) slot_of[wave][0] = 0;
  }
  {
    int to[5], from[4];
#pragma unroll
    for (int r = 0; r < 5; ++r) to[r] = __builtin_amdgcn_readlane(ends, 4 * wave + r);
#pragma unroll
    for (int r = 0; r < 4; ++r) from[r] = (4 * wave + r) * kSmallTile + __builtin_amdgcn_readlane(lb, 4 * wave + r) - to[r];
    for (int i0 = to[0] + lane; i0 - lane < to[4]; i0 += 8 * 64) {
      uint64_t w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = min(i0 + e * 64, to[4] - 1);
        w[e] = in[i + (i >= to[3] ? from[3] : i >= to[2] ? from[2] : i >= to[1] ? from[1] : from[0])];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (i0 + e * 64 < to[4]) buf[at(i0 + e * 64)] = to_double(w[e]);
    }
  }
  __syncthreads();

  // ---- pairwise merges in LDS.  A slot's eight outputs start at a point of the merge path; they are the smaller ones of
  // the next eight words of one run, ascending, and the next eight of the other, descending, a bitonic sequence that three
  // steps put in order: all sixteen reads are in flight together, where merging word by word waits for each.
  const int runs = (n_group + kSmallTile - 1) / kSmallTile;
#pragma unroll 1
  for (int level = 0; 1 << level < runs; ++level) {
    const int* slots = slot_of[level];
    const int used = __builtin_amdgcn_readfirstlane(slots[kCutRuns / 2 >> level]);
    double res[2][kCutItems];
    int to[2], count[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int slot = t + e * kCutThreads;
      count[e] = 0;
      if (e * kCutThreads + (t & ~63) >= used) continue;     // uniform over the wave
      int q = 0;
      for (int step = kCutRuns / 4 >> level; step > 0; step >>= 1)
        if (slots[q + step] <= slot) q += step;
      const int b0 = start_of[q << (level + 1)], mid = start_of[(2 * q + 1) << level], end = start_of[(q + 1) << (level + 1)];
      const int d0 = min((slot - slots[q]) * kCutItems, end - b0);
      const int x = merge_path_lds<kCutItems>(buf, b0, mid - b0, mid, end - mid, d0);
      const int ia = b0 + x, ib = mid + d0 - x;
      double o[kCutItems];
#pragma unroll
      for (int i = 0; i < kCutItems; ++i) {
        res[e][i] = buf[at(ia + i)];
        o[i] = buf[at(ib + i)];
      }
      if (__builtin_amdgcn_ballot_w64(ia + kCutItems > mid || ib + kCutItems > end) != 0) {
#pragma unroll
        for (int i = 0; i < kCutItems; ++i) {
          if (ia + i >= mid) res[e][i] = INFINITY;
          if (ib + i >= end) o[i] = INFINITY;
        }
      }
#pragma unroll
      for (int i = 0; i < kCutItems; ++i) res[e][i] = min_of(res[e][i], o[kCutItems - 1 - i]);
#pragma unroll
      for (int step = kCutItems / 2; step > 0; step >>= 1)
#pragma unroll
        for (int i = 0; i < kCutItems; ++i) {
          if (i & step) continue;
          const double v = res[e][i], w = res[e][i + step];
          res[e][i] = min_of(v, w);
          res[e][i + step] = max_of(v, w);
        }
      to[e] = b0 + d0;
      count[e] = min(kCutItems, end - b0 - d0);
    }
    __syncthreads();                         // everyone is done reading the pieces
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int i = 0; i < kCutItems; ++i)
        if (i < count[e]) buf[at(to[e] + i)] = res[e][i];
    __syncthreads();
  }
  int32_t* perm_out = bh < a.BH0 ? a.perm0 : (a.perm1 ? a.perm1 - (int64_t)a.BH0 * g.L : nullptr);
  const int64_t obase = (int64_t)bh * g.L + a0 + base;
  if (perm_out) {
    for (int i = t; i < n; i += kCutThreads) perm_out[obase + i] = idx_of_double(buf[at(i)]);
  } else {
    for (int i = t; i < n; i += kCutThreads) a.out[obase + i] = to_word(buf[at(i)]);
  }
}
__global__ __launch_bounds__(kCutThreads) void cut_merge_kernel(CutArgs a) {
  const int total = gridDim.x;             // a head's words on one XCD
  cut_merge(a, (total & 7) == 0 ? (blockIdx.x & 7) * (total >> 3) + (blockIdx.x >> 3) : blockIdx.x);
}
struct CutJob {
  CutArgs a;
  __device__ __forceinline__ void run(int block) const { cut_merge(a, block); }
};

__global__ void iota_kernel(int32_t* perm, int L, int64_t total) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) perm[i] = (int32_t)(i % L);
}

}  // namespace

size_t sort_workspace_bytes(int BH, int L) {
  return 2 * align_up((size_t)BH * L * sizeof(uint64_t), 256);
}

basa_status launch_iota_perm(int32_t* perm, int BH, int L, hipStream_t st) {
  int64_t total = (int64_t)BH * L;
  if (total == 0) return BASA_OK;
  hipLaunchKernelGGL(iota_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, perm, L, total);
  BASA_HIP_CHECK_LAUNCH("iota_kernel");
  return BASA_OK;
}

static SegGeom geom_of(int L, int window, int tile) {
  SegGeom g;
  g.L = L;
  g.W = (window > 0 && window < L) ? window : L;      // a segment list is sorted as one run of L
  g.segs = ceil_div(L, g.W);
  g.tiles_per_seg = ceil_div(g.W, tile);
  return g;
}

// Is a call's first merge the one that is cut by sampling?  Few words: from 3 x 2^17 on, where ranking takes two passes (sort,
// ranking / cut: 8 rows of 32768: 39.5 / 40.1 us, 10: 51.6 / 49.1, 16: 66.4 / 53.3, 24 of 16384: 48.0 / 47.8, 32: 56.2 / 51.3).  More: wherever
// runs have more than two tiles (quads of 16384 words in LDS and merge passes / cut: 64 rows of 32768 149 / 142, 32: 101 / 84, 64 of
// 16384: 87 / 77, 64 of 8200: 78 / 62, 8 of 100000: 128 / 100).
static bool cut_pays(int run, int64_t words, bool few) {
  return few ? run > 8 * kSmallTile && words >= 3 << 17 : run > 2 * kSmallTile;
}
// Parts of 2048 words, of 3072 where those would be more than three to a compute unit (64 rows of 32768: 148 / 143 us; 40: 103 / 97,
// 32: 83.5 / 84.6, 48 of 16384: 66 / 69).  Runs of up to 4096 words (packed batches) in one part of 3072 or two of 2048: a second part of
// what is left takes as long as the first.  Merge, by the line of the others / this: 32 heads on 8, 11 sequences of 2065 to
// 2246: 29.1 / 17.9 us, 32 on 32, 11 of 2060 to 2273: 35.6 / 20.6, 11 of 2738 to 3370: 40.7 / 36.1, 9 of 3921 to 4089: 43.0 / 35.0.
static CutArgs cut_args(const uint64_t* src, uint64_t* dst, int32_t* perm0, int32_t* perm1, int BH0, const SegGeom& g, int64_t words) {
  const bool large = g.W > 2 * kPartSamples * kCutStride ? words > (int64_t)3 * 256 * kPartSamples * kCutStride : g.W <= kMaxPartSamples * kCutStride;
  const int samples = large ? kMaxPartSamples : kPartSamples;
  return CutArgs{src, dst, perm0, perm1, BH0, g, ceil_div(g.W, kCutWords), ceil_div(std::min(g.W, kCutWords), samples * kCutStride), samples};
}

// Sorted tiles in src merged into whole segments: BH rows (the first BH0 go to perm0, the rest to perm1).
static basa_status merge_tiles(uint64_t* src, uint64_t* dst, int BH, int BH0, const SegGeom& g, int tile, bool few,
                               int32_t* perm0, int32_t* perm1, hipStream_t st) {
  const int L = g.L;
  int64_t sorted = tile;                       // words of a run
  if (tile == kSmallTile && cut_pays(g.W, (int64_t)BH * L, few)) {
    const bool last = g.W <= kCutWords;
    const CutArgs args = cut_args(src, dst, last ? perm0 : nullptr, last ? perm1 : nullptr, BH0, g, (int64_t)BH * L);
    ProfScope prof(K_MERGE, st);
    hipLaunchKernelGGL(cut_merge_kernel, dim3((unsigned)(BH * g.segs * args.groups_per_seg * args.parts)), dim3(kCutThreads), 0, st, args);
    BASA_HIP_CHECK_LAUNCH("cut_merge_kernel");
    uint64_t* t = src; src = dst; dst = t;
    sorted = kCutWords;
  }
  if (few) {
    // as few passes as groups of up to eight runs allow, each with the smallest group that keeps to that number
    const int chunks = ceil_div(L, kSortThreads);
    int passes = 0;
    for (int64_t r = 1; r < (g.W + sorted - 1) / sorted; r *= 8) ++passes;
    for (int64_t run = sorted; run < g.W; --passes) {
      const int64_t runs = (g.W + run - 1) / run;
      int G = 2;
      while (G < 8 && (passes == 1 ? G : passes == 2 ? G * G : (int64_t)G * G * G) < runs) G *= 2;
      const bool last = run * G >= g.W;
      ProfScope prof(K_MERGE, st);
      const RankArgs args{src, dst, last ? perm0 : nullptr, last ? perm1 : nullptr, BH0, g, (int)run, chunks};
#define BASA_RANK(N) \
  hipLaunchKernelGGL((rank_runs_kernel<N, RankArgs>), dim3((unsigned)chunks * BH), dim3(kSortThreads), 0, st, args)
      if (G == 2) BASA_RANK(2);
      else if (G == 4) BASA_RANK(4);
      else BASA_RANK(8);
#undef BASA_RANK
      BASA_HIP_CHECK_LAUNCH("rank_runs_kernel");
      uint64_t* t = src; src = dst; dst = t;
      run *= G;
    }
    return BASA_OK;
  }
  int run0 = (int)sorted;
  if (sorted == kTile && g.W > 2 * kTile) {
    // more than two tiles per segment: the first two passes in one launch
    const bool last = kQuadWords >= g.W;
    const int quads_per_seg = ceil_div(g.W, kQuadWords);
    const int quads_total = BH * g.segs * quads_per_seg;
    // one quad per workgroup while there are compute units for all (64 quads: 21.7 us, two per workgroup 37)
    const int quad_wgs = quads_total <= 512 ? std::min(quads_total, 256) : ceil_div(quads_total, 2);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&merge_quads_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kQuadWords * 8);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");
    ProfScope prof(K_MERGE, st);
    hipLaunchKernelGGL(merge_quads_kernel, dim3(quad_wgs), dim3(kQuadThreads), kQuadWords * 8, st, src, dst,
                       last ? perm0 : nullptr, last ? perm1 : nullptr, BH0, g, quads_per_seg, quads_total);
    BASA_HIP_CHECK_LAUNCH("merge_quads_kernel");
    uint64_t* t = src; src = dst; dst = t;
    run0 = kQuadWords;
  }
  for (int run = run0; run < g.W; run *= 2) {
    const bool last = run * 2 >= g.W;
    const int pairs_per_seg = ceil_div(ceil_div(g.W, run), 2);
    const int chunks_per_pair = ceil_div(2 * run, kMergeChunk);
    ProfScope prof(K_MERGE, st);
    hipLaunchKernelGGL(merge_pass_kernel, dim3(g.segs * pairs_per_seg * chunks_per_pair, BH),
                       dim3(kSortThreads), 0, st, src, dst, last ? perm0 : nullptr, last ? perm1 : nullptr,
                       BH0, g, run, chunks_per_pair, pairs_per_seg);
    BASA_HIP_CHECK_LAUNCH("merge_pass_kernel");
    uint64_t* t = src; src = dst; dst = t;
  }
  return BASA_OK;
}

// Sort one tensor (x1 == nullptr) or two tensors of identical d and dtype in the same launches.
static basa_status norm_sort_impl(const TensorView& x0, const TensorView* x1, int window, const SegList& segs, int32_t* perm0,
                                  int32_t* perm1, float* keys_out, void* ws, bool cached, hipStream_t st) {
  const int BH0 = x0.batch * x0.heads, BH1 = x1 ? x1->batch * x1->heads : 0, L0 = x0.L, L1 = x1 ? x1->L : x0.L;
  const int64_t words0 = (int64_t)BH0 * L0, words = words0 + (int64_t)BH1 * L1;
  if (words == 0) return BASA_OK;
  const SortPlan plan = plan_sort(BH0, L0, BH1, L1, window, x0.d * (x0.dtype == BASA_BF16 ? 2 : 4), cached);
  const bool few = plan.few;
  const int tile = plan.tile;
  if (x1 && ((L0 != L1 && !few) || BH0 + BH1 > 65535)) {       // (65535: the grid's second dimension)
    const basa_status s = norm_sort_impl(x0, nullptr, window, segs, perm0, nullptr, keys_out, ws, cached, st);
    return s != BASA_OK ? s : norm_sort_impl(*x1, nullptr, window, segs, perm1, nullptr, nullptr, ws, cached, st);
  }
  uint64_t* buf0 = reinterpret_cast<uint64_t*>(ws);
  uint64_t* buf1 = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(ws) + align_up((size_t)words * sizeof(uint64_t), 256));
  const TensorView& xb = x1 ? *x1 : x0;
  const bool bf16 = x0.dtype == BASA_BF16;
  const SegGeom g0 = geom_of(L0, window, tile), g1 = geom_of(L1, window, tile);
  const bool single0 = g0.tiles_per_seg == 1, single1 = g1.tiles_per_seg == 1;
  {
  ProfScope prof(K_NORM_TILE_SORT, st);
  // With different lengths a grid of the longer one's tiles by rows would be mostly workgroups that return at once, and which
  // compute units get two real ones is then a matter of their timing: 256 queries of 32768, 32 heads on 8: 34 to 42 us, 24 in one row.
  const int per0 = g0.segs * g0.tiles_per_seg, per1 = g1.segs * g1.tiles_per_seg;
  const int tiles1 = x1 && L0 != L1 ? BH1 * per1 : 0;
  // Eight waves to a tile instead of four where the tiles leave compute units idle: twice the rows in flight in each, half the words
  // to a lane.  Sort, four -> eight waves: 2 fp32 rows of 1024, d = 64: 12.9 -> 11.7 us, 64 of 512: 13.8 -> 11.2; tiles of 512: 40 of 2000:
  // 15.3 -> 12.2, 16 of 2472: 15.9 -> 12.7; level at 160 tiles of 1024 and kept at four beyond 128: 192: 27.5 / 28.1, 256: 39.8 / 43.3;
  // fp32, d = 128, 128 tiles of 512: the whole operator 213.8 / 215.6.
  const int tiles = per0 * BH0 + per1 * BH1, token_bytes = x0.d * (bf16 ? 2 : 4);
  const bool eight = tile == kSmallTile ? tiles <= 128 : tiles * token_bytes <= 48 * 1024;
  const dim3 grid = tiles1 > 0 ? dim3(BH0 * per0 + tiles1) : dim3(per0, BH0 + BH1);
#define BASA_KEYS_T(BF, D, T, S, N)                                                                            \
  hipLaunchKernelGGL((norm_tile_sort_kernel<BF, D, T, N, S>), grid, dim3(N), 0, st, x0, xb, BH0, buf1, \
                     single0 ? perm0 : nullptr, single1 ? perm1 : nullptr, keys_out, g0, g1, segs, tiles1)
#define BASA_KEYS(BF, D)                                                                   \
  do {                                                                                     \
    if (tile == kTile && !cached) BASA_KEYS_T(BF, D, kTile, true, kSortThreads);           \
    else if (tile == kTile) BASA_KEYS_T(BF, D, kTile, false, kSortThreads);                \
    else if (!cached) BASA_KEYS_T(BF, D, kSmallTile, true, kSortThreads);                  \
    else if (tile == 512 && eight) BASA_KEYS_T(BF, D, 512, false, 2 * kSortThreads);       \
    else if (tile == 512) BASA_KEYS_T(BF, D, 512, false, kSortThreads);                    \
    else if (eight) BASA_KEYS_T(BF, D, kSmallTile, false, 2 * kSortThreads);               \
    else BASA_KEYS_T(BF, D, kSmallTile, false, kSortThreads);                              \
  } while (0)
  if (bf16 && x0.d == 128) BASA_KEYS(true, 128);
  else if (bf16 && x0.d == 64) BASA_KEYS(true, 64);
  else if (!bf16 && x0.d == 128) BASA_KEYS(false, 128);
  else BASA_KEYS(false, 64);
#undef BASA_KEYS
#undef BASA_KEYS_T
  BASA_HIP_CHECK_LAUNCH("norm_tile_sort_kernel");
  }
  if (L0 == L1) return single0 ? BASA_OK : merge_tiles(buf1, buf0, BH0 + BH1, BH0, g0, tile, few, perm0, perm1, st);
  basa_status s = BASA_OK;
  if (!single0) s = merge_tiles(buf1, buf0, BH0, BH0, g0, tile, few, perm0, nullptr, st);
  if (s == BASA_OK && !single1) s = merge_tiles(buf1 + words0, buf0 + words0, BH1, BH1, g1, tile, few, perm1, nullptr, st);
  return s;
}

template <int kG>
static basa_status rank_many(const SeqJob* seq, int n, int run, int pass, hipStream_t st) {
  Jobs<RankArgs> jobs;
  for (int i = 0; i < n; ++i) {
    const int L = seq[i].q.L, rows = seq[i].q.heads + seq[i].k.heads;
    if (run >= L) continue;                                // sorted by an earlier pass
    const bool last = (int64_t)run * kG >= L;
    uint64_t* buf[2] = {reinterpret_cast<uint64_t*>(seq[i].sort_ws),
                        reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(seq[i].sort_ws) + align_up((size_t)rows * L * 8, 256))};
    jobs.add(RankArgs{buf[pass & 1], buf[(pass & 1) ^ 1], last ? seq[i].perm_q : nullptr, last ? seq[i].perm_k : nullptr,
                      seq[i].q.heads, geom_of(L, 0, kSmallTile), run, ceil_div(L, kSortThreads)},
             (int64_t)ceil_div(L, kSortThreads) * rows);
  }
  if (jobs.n == 0) return BASA_OK;
  ProfScope prof(K_MERGE, st);
  hipLaunchKernelGGL((rank_runs_kernel<kG, Jobs<RankArgs>>), dim3(jobs.first[jobs.n]), dim3(kSortThreads), 0, st, jobs);
  BASA_HIP_CHECK_LAUNCH("rank_runs");
  return BASA_OK;
}
template <int kD>
static basa_status sort_many(const SeqJob* seq, int n, hipStream_t st) {
  int longest = 0;
  {
    Jobs<SmallSortJob<kD>> jobs;
    for (int i = 0; i < n; ++i) {
      const SegGeom g = geom_of(seq[i].q.L, 0, kSmallTile);
      const bool single = g.tiles_per_seg == 1;
      jobs.add(SmallSortJob<kD>{seq[i].q, seq[i].k, reinterpret_cast<uint64_t*>(seq[i].sort_ws), single ? seq[i].perm_q : nullptr,
                                single ? seq[i].perm_k : nullptr, g},
               (int64_t)g.tiles_per_seg * (seq[i].q.heads + seq[i].k.heads));
      longest = std::max(longest, seq[i].q.L);
    }
    ProfScope prof(K_NORM_TILE_SORT, st);
    hipLaunchKernelGGL(many_kernel<SmallSortJob<kD>>, dim3(jobs.first[n]), dim3(kSortThreads), 0, st, jobs);
    BASA_HIP_CHECK_LAUNCH("norm_tile_sort");
  }
  // Cut by samples, or ranked: from 3 x 2^17 words on, where ranking takes two passes or a pass of eight runs; of four runs, three or four
  // of which are used, from 3 x 2^18 on; sequences longer than a group are ranked.  Merge, rank / cut: 16 heads on 16, 4 of 3928 to 4054
  // tokens (0.51 million words): 11.8 / 15.7 us; 32 on 8, 8 of 2113 to 2289 (0.72): 16.4 / 17.2; 32 on 32, 6 of 2141 to 2188 (0.83): 18.2 / 17.4, 8 of
  // 2066 to 2273 (1.11): 23.0 / 18.0; two used: 32 on 32, 6 of 1217 to 2035 (0.60): 14.5 / 11.9; eight: 32 on 8, 2 of 5341 to 5813 (0.45): 20.0 / 17.6.
  int64_t words = 0;
  for (int i = 0; i < n; ++i) words += seq[i].q.L > kSmallTile ? (int64_t)seq[i].q.L * (seq[i].q.heads + seq[i].k.heads) : 0;
  const bool four_used = longest > 2 * kSmallTile && longest <= 4 * kSmallTile;
  if (words >= (four_used ? 3 << 18 : 3 << 17) && longest <= kCutWords) {
    Jobs<CutJob> jobs;
    for (int i = 0; i < n; ++i) {
      const int L = seq[i].q.L, rows = seq[i].q.heads + seq[i].k.heads;
      if (L <= kSmallTile) continue;
      uint64_t* src = reinterpret_cast<uint64_t*>(seq[i].sort_ws);
      const CutArgs a = cut_args(src, nullptr, seq[i].perm_q, seq[i].perm_k, seq[i].q.heads, geom_of(L, 0, kSmallTile), words);
      jobs.add(CutJob{a}, (int64_t)a.parts * rows);
    }
    ProfScope prof(K_MERGE, st);
    hipLaunchKernelGGL((many_kernel<CutJob, 1, kCutThreads>), dim3(jobs.first[jobs.n]), dim3(kCutThreads), 0, st, jobs);
    BASA_HIP_CHECK_LAUNCH("cut_merge");
    return BASA_OK;
  }
  // groups of eight runs (four if that is enough) until the longest sequence is one run
  int pass = 0;
  for (int64_t run = kSmallTile; run < longest; ++pass) {
    const bool four = run * 4 >= longest;
    const basa_status s = four ? rank_many<4>(seq, n, (int)run, pass, st) : rank_many<8>(seq, n, (int)run, pass, st);
    if (s != BASA_OK) return s;
    run *= four ? 4 : 8;
  }
  return BASA_OK;
}
basa_status launch_norm_sort_many(const SeqJob* seq, int n, hipStream_t st) {
  return seq[0].q.d == 128 ? sort_many<128>(seq, n, st) : sort_many<64>(seq, n, st);
}

basa_status launch_norm_sort(const TensorView& x, int window, const SegList& segs, int32_t* perm, float* keys_out,
                             void* ws, bool cached, hipStream_t st) {
  return norm_sort_impl(x, nullptr, window, segs, perm, nullptr, keys_out, ws, cached, st);
}

basa_status launch_norm_sort2(const TensorView& q, const TensorView& k, int window, const SegList& segs,
                              int32_t* perm_q, int32_t* perm_k, void* ws, bool cached, hipStream_t st) {
  return norm_sort_impl(q, &k, window, segs, perm_q, perm_k, nullptr, ws, cached, st);
}

}  // namespace basa
