// Block-sparse attention on the bf16 matrix cores of gfx950 (Sec. 2; Eq. 1; Alg. 1
// step 12), head dimension D = 128 (the shapes below) or 64 (rows, tiles and accumulators
// half as large: 8 chunks per row, K swizzle by row & 7, 8 KB tiles).
//
// Layout prepared once per call by the gather kernels below (workspace).  K and V are
// stored as 64-key tiles that are byte-for-byte the LDS image the main kernel wants, so
// the global -> LDS copy is a linear 16 KB copy done with direct-to-LDS loads:
//   (Q needs no copy: every wave reads the rows of its 32 queries once, through perm_q)
//   Kt [BHkv][tiles][64 rows][16 chunks of 8 bf16]   rows of K in sorted order; chunk c
//        of row r sits at chunk position c ^ (r & 15)                (XOR swizzle)
//   Vt [BHkv][tiles][128 d-rows][8 chunks of 8 keys] V in sorted order, transposed per
//        tile (d major); the 8 keys of a chunk are in MFMA operand-slot order (below);
//        chunk c of d-row r sits at chunk position c ^ ((r >> 1) & 7)
// The swizzles make every ds_read_b128 of 16 consecutive lanes hit 16 distinct 16-byte
// bank groups.  Calls of few queries have no such copy (attn_rows.hpp): the 128-query shape fetches the rows of K and V
// from the caller's tensors, through perm_k, into the same K image and an image of V by rows, from which a
// transposing LDS read takes V^T.
//
// Main kernel: a workgroup owns 512, 256 or 128 consecutive sorted queries, i.e. 4, 2 or 1 query blocks of 128
// (twice as many of 64); a wave owns 64 queries in the first shape, which large calls run on, and 32 in the
// others (see kWideQueries below).  Streaming K/V tiles from L2 into LDS is the costly part beside the MFMAs
// themselves, so the query blocks of a workgroup share every tile: it walks the UNION of their block lists in
// ascending order, each tile is fetched once, and only the waves whose query block lists the tile's key block
// compute on it.  Scores are computed TRANSPOSED, S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16 (A = K tile rows from LDS, B = Q^T held in registers), so that every lane owns ONE query: the running max,
// running sum and the rescale factor of the online softmax are per-lane scalars, the
// row max needs a single exchange between lanes l and l+32, and the exponentiated
// accumulator registers are, after packing to bf16, already the B operand of the
// second product O^T = V^T P^T (A = V^T tile rows from LDS).
// The accumulator of a 32x32 MFMA holds, in lane half h, rows 4h+{0..3} and 8+4h+{0..3}
// of each 16-row group; packing those 8 values gives operand slot 8h+e <-> key
// 8*(e/4) + 4h + e%4 of the group, which is the key order inside a Vt chunk pair.
// The running max is refreshed lazily: the accumulators are rescaled only when some
// query's tile max exceeds its running max by more than 2^8, so the common iteration
// touches O only through MFMA (or there is no running max at all, see process_tile2).  K/V tiles go
// through an LDS ring: two stages and a workgroup barrier per tile in the 128-query shape, two slots of two
// tiles in the 256-query one, up to four stages in the 512-query one, whose query blocks may be at different tiles.
#include <algorithm>
#include <climits>
#include <cmath>
#include <type_traits>
#include "attn_lds.hpp"
#include "attn_rows.hpp"
#include "common.hpp"

namespace basa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));

constexpr float kLazyTau = 8.0f;            // log2 of the largest exponentiated score kept
// Running maximum (log2 units) of a query that has met no score above -inf yet: below every finite one (a float times
// log2(e) / 8 at most), and itself finite, so that its scores of -inf exponentiate to 0 and rescaling it by itself is 1;
// from -inf both would be exp2(inf - inf).
constexpr float kNoMax = -1e38f;
// The pass without running maxima (64 queries per wave): a query's reference moves up by kShiftLog2
// once the probabilities of half a tile add up to more than kSafeSum; a row whose final sum lies
// outside [kMinSum, kMaxSum] (or is not a number) has left the range in which that pass is exact.
constexpr float kSafeSum = 1.0995116e12f;   // 2^40
constexpr float kShiftLog2 = 40.0f;
constexpr float kShiftMul = 9.094947e-13f;  // 2^-40
constexpr float kMinSum = 8.6736174e-19f;   // 2^-60
constexpr float kMaxSum = 1.2676506e30f;    // 2^100
// Two shapes of workgroup.  SHARED: 8 waves own 256 queries = two (four) neighbouring query blocks
// that share every K/V tile; best when their lists overlap, which they do for the full method.
// SOLO: 4 waves own 128 queries = one query block of 128 (two of 64), two workgroups per compute
// unit; every tile is fetched per 128 queries, but no wave ever waits for a tile that only its
// neighbour lists - best when neighbouring lists have little in common.
constexpr int kSharedQueries = 256, kSoloQueries = 128, kWideQueries = 512;
#ifndef BASA_ATTN_DEFAULT_LISTS
#define BASA_ATTN_DEFAULT_LISTS 3      // shape taken for block lists the overlap probe does not cover
#endif

// ---------------------------------------------------------------------------------
// Gather kernels
// ---------------------------------------------------------------------------------
// Rows of a tile given by a table of row indices (INT_MAX: no row, zeros).  As in gather_chunks, all loads are
// unconditional and in flight together.
template <int ITERS>
__device__ __forceinline__ void gather_listed(uint4 (&v)[ITERS], const int* rows, const char* base, int L, int64_t row_bytes,
                                              int first, int step, int sub) {
  int row[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) row[it] = rows[first + it * step];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) v[it] = reinterpret_cast<const uint4*>(base + min(row[it], L - 1) * row_bytes)[sub];
#pragma unroll
  for (int it = 0; it < ITERS; ++it)
    if (row[it] == INT_MAX) v[it] = make_uint4(0u, 0u, 0u, 0u);
}

// 64 rows of K in sorted order, zero-padded, in K-tile order (rows: the rows of the tile, or null for perm's order).
template <int D>
__device__ __forceinline__ void gather_k_tile(const TensorView& x, const int32_t* __restrict__ pm, const int* rows,
                                              uint4* __restrict__ dst, int bh, int tile, int tiles_per_head) {
  constexpr int CPR = Geo<D>::kChunksPerRow, RPI = 256 / CPR, ITERS = 64 / RPI;
  const int sub = threadIdx.x % CPR, rig = threadIdx.x / CPR;
  const char* base = reinterpret_cast<const char*>(x.ptr) + x.head_offset(bh) * 2;
  uint4 v[ITERS];
  if (rows) gather_listed<ITERS>(v, rows, base, x.L, (int64_t)x.stride_l * 2, rig, RPI, sub);
  else gather_chunks<ITERS>(v, pm, base, x.L, (int64_t)x.stride_l * 2, tile * kTileKeys + rig, RPI, sub);
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int pos = tile * kTileKeys + it * RPI + rig;
    dst[((int64_t)bh * tiles_per_head * kTileKeys + pos) * CPR + (sub ^ (pos & (CPR - 1)))] = v[it];
  }
}

// V: gather 64 sorted rows, transpose through LDS, write the swizzled [D][64] tile.
template <int D>
__device__ __forceinline__ void gather_vt_tile(const TensorView& v, const int32_t* __restrict__ pm, const int* listed,
                                               uint4* __restrict__ dst, int bh, int tile, int tiles_per_head) {
  constexpr int CPR = Geo<D>::kChunksPerRow, RPI = 256 / CPR, ITERS = 64 / RPI;
  constexpr int kRowStride = D + 8;   // one row + 16 B pad
  __shared__ __attribute__((aligned(16))) uint16_t rows[kTileKeys][kRowStride];
  const int sub = threadIdx.x % CPR, rig = threadIdx.x / CPR;
  const char* base = reinterpret_cast<const char*>(v.ptr) + v.head_offset(bh) * 2;
  uint4 val[ITERS];
  if (listed) gather_listed<ITERS>(val, listed, base, v.L, (int64_t)v.stride_l * 2, rig, RPI, sub);
  else gather_chunks<ITERS>(val, pm, base, v.L, (int64_t)v.stride_l * 2, tile * kTileKeys + rig, RPI, sub);
#pragma unroll
  for (int it = 0; it < ITERS; ++it) *reinterpret_cast<uint4*>(&rows[it * RPI + rig][sub * 8]) = val[it];
  __syncthreads();
  // 8 D output chunks of 8 slots; thread handles chunk (d = id/8, s8 = id%8):
  // 16-key group g16 = s8/2, lane half hh = s8%2, slot e <-> key 16 g16 + 8(e/4) + 4 hh + e%4
#pragma unroll
  for (int it = 0; it < D * 8 / 256; ++it) {
    const int id = it * 256 + threadIdx.x;
    const int dd = id >> 3, s8 = id & 7;
    const int g16 = s8 >> 1, hh = s8 & 1;
    uint16_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int key = 16 * g16 + 8 * (j >> 2) + 4 * hh + (j & 3);
      e[j] = rows[key][dd];
    }
    uint4 o;
    o.x = e[0] | ((uint32_t)e[1] << 16); o.y = e[2] | ((uint32_t)e[3] << 16);
    o.z = e[4] | ((uint32_t)e[5] << 16); o.w = e[6] | ((uint32_t)e[7] << 16);
    dst[(((int64_t)bh * tiles_per_head + tile) * D + dd) * 8 + (s8 ^ ((dd >> 1) & 7))] = o;
  }
}

// Causal variant: the original index of every key of a tile (INT_MAX past the end of the sequence), then the smallest
// of all, the smallest of the second 32, the largest of the first 32 and of the second 32.
__device__ __forceinline__ void key_index_tile(const int32_t* __restrict__ pm, const int* rows, int Lk, int32_t* __restrict__ out,
                                               int bh, int tile, int tiles_per_head) {
  const int lane = threadIdx.x;
  if (lane >= 64) return;
  const int pos = tile * kTileKeys + lane;
  const int idx = rows ? rows[lane] : pos < Lk ? perm_at(pm, 0, pos, Lk) : INT_MAX;
  int lo = idx, hi = idx;
#pragma unroll
  for (int off = 16; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off));
    hi = max(hi, __shfl_xor(hi, off));
  }
  const int lo_other = __shfl_xor(lo, 32);
  int32_t* o = out + ((int64_t)bh * tiles_per_head + tile) * kIxStride;
  o[lane] = idx;
  if (lane == 0) { o[kTileKeys] = min(lo, lo_other); o[kTileKeys + 1] = lo_other; o[kTileKeys + 2] = hi; }
  if (lane == 32) o[kTileKeys + 3] = hi;
}

// The entries of `raw` (128 of them, a block's original indices; INT_MAX where there is none) by increasing value, entry
// t placed by thread t: its place is the number of entries before it.
__device__ __forceinline__ int place_in_block(const int* raw, int t) {
  const int mine = raw[t];
  int place = 0;
#pragma unroll 8
  for (int j = 0; j < 128; j += 4) {
    const int4 x = *reinterpret_cast<const int4*>(raw + j);
    place += (x.x < mine || (x.x == mine && j < t)) + (x.y < mine || (x.y == mine && j + 1 < t)) +
             (x.z < mine || (x.z == mine && j + 2 < t)) + (x.w < mine || (x.w == mine && j + 3 < t));
  }
  return place;
}

// Which key blocks the lists of a KV head name, as bitmaps [BHkv][parts][ceil(Nk / 32)], one workgroup to a part (a run
// of the rows of the `rows` lists of the KV head's query heads, which are neighbours): the blocks that nobody lists
// need no tiles.  The rows agree in much of what they keep: 19 % of the blocks are listed by any of 128 rows that keep
// 10 % each, 40 % at 25 %, 68 % at 50 % (L = 16384).  An entry is one independent load per thread, four in flight.
constexpr int kMaxListedWords = 512;         // 16384 key blocks: more than the main kernel lists
constexpr int kListedParts = 16;
__global__ __launch_bounds__(1024) void listed_blocks_kernel(const int32_t* __restrict__ row_count,
                                                             const int32_t* __restrict__ row_cols, int cols_stride, int rows,
                                                             int Nk, uint32_t* __restrict__ listed) {
  __shared__ uint32_t bits[kMaxListedWords];
  const int words = (Nk + 31) >> 5, parts = gridDim.y, part = blockIdx.y;
  for (int w = threadIdx.x; w < words; w += 1024) bits[w] = 0u;
  __syncthreads();
  const int r0 = (int)((int64_t)rows * part / parts), r1 = (int)((int64_t)rows * (part + 1) / parts);
  const int64_t row0 = (int64_t)blockIdx.x * rows + r0, entries = (int64_t)(r1 - r0) * cols_stride;
  for (int64_t e0 = threadIdx.x; e0 < entries; e0 += 4 * 1024) {
    unsigned col[4];
    int left[4];                             // entries of the row from this one on
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t e = min(e0 + u * 1024, entries - 1);       // (past the end: the last one again)
      const int r = (int)((uint32_t)e / (uint32_t)cols_stride), i = (int)e - r * cols_stride;
      left[u] = row_count[row0 + r] - i;
      col[u] = (unsigned)row_cols[row0 * cols_stride + e];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (left[u] > 0 && col[u] < (unsigned)Nk) atomicOr(&bits[col[u] >> 5], 1u << (col[u] & 31));
  }
  __syncthreads();
  for (int w = threadIdx.x; w < words; w += 1024) listed[((int64_t)blockIdx.x * parts + part) * words + w] = bits[w];
}

// Everything the main kernel reads besides Q, in one launch (small calls pay about 4 us for each): blockIdx.z = 0 the
// K tiles and (causal) the key indices, 1 the V^T tiles; the counters of the overlap probe start at zero.
// by_index (causal, blocks of 128): the keys of a block in the order of their original indices instead of perm's.  A
// list names whole blocks, so the order inside one is free, and this one lets the main kernel leave out the half
// tiles whose keys all come after a wave's queries.
template <int D>
__device__ __forceinline__ void tile_kv(int tile, int bh, bool is_v, int tiles_per_head, const TensorView& k, const TensorView& v,
                                        const int32_t* __restrict__ perm, uint4* __restrict__ Kt, uint4* __restrict__ Vt,
                                        int32_t* __restrict__ kix, int32_t* __restrict__ probe, int by_index,
                                        const uint32_t* __restrict__ listed, int parts, int tiles_per_block) {
  __shared__ __attribute__((aligned(16))) int raw[128], ordered[128], place[128];
  const int32_t* pm = perm ? perm + (int64_t)bh * k.L : nullptr;
  const int* rows = nullptr;
  if (probe && !is_v && tile == 0 && bh == 0 && threadIdx.x < 2) probe[threadIdx.x] = 0;
  if (listed) {                                      // uniform: nobody reads the tiles of a block in no list
    const int block = tile / tiles_per_block, words = (tiles_per_head / tiles_per_block + 31) >> 5;
    uint32_t any = 0u;
    for (int p = 0; p < parts; ++p) any |= listed[((int64_t)bh * parts + p) * words + (block >> 5)];
    if (!((any >> (block & 31)) & 1u)) return;
  }
  if (by_index) {
    // ranked by counting, two threads to an entry (places past the keys, and those a malformed perm leaves open, stay
    // without a row)
    constexpr int kNone = INT_MAX - 127;
    const int t = threadIdx.x, e = t & 127, pos = (tile >> 1) * 128 + e;
    if (t < 128) {
      raw[t] = pos < k.L ? perm_at(pm, 0, pos, k.L) : kNone + t;
      ordered[t] = INT_MAX;
      place[t] = 0;
    }
    __syncthreads();
    const int mine = raw[e];
    int before = 0;
#pragma unroll
    for (int j = 0; j < 64; j += 4) {
      const int4 x = *reinterpret_cast<const int4*>(raw + (t >> 7) * 64 + j);
      before += (x.x < mine) + (x.y < mine) + (x.z < mine) + (x.w < mine);
    }
    atomicAdd(&place[e], before);
    __syncthreads();
    if (t < 128 && mine < kNone) ordered[place[t]] = mine;
    __syncthreads();
    rows = ordered + (tile & 1) * kTileKeys;
  }
  if (!is_v) {
    gather_k_tile<D>(k, pm, rows, Kt, bh, tile, tiles_per_head);
    if (kix) key_index_tile(pm, rows, k.L, kix, bh, tile, tiles_per_head);
  } else {
    gather_vt_tile<D>(v, pm, rows, Vt, bh, tile, tiles_per_head);
  }
}

template <int D>
__global__ __launch_bounds__(256) void tile_kv_kernel(TensorView k, TensorView v, const int32_t* __restrict__ perm,
                                                      uint4* __restrict__ Kt, uint4* __restrict__ Vt, int32_t* __restrict__ kix,
                                                      int32_t* __restrict__ probe, int by_index,
                                                      const uint32_t* __restrict__ listed, int parts, int tiles_per_block) {
  tile_kv<D>(blockIdx.x, blockIdx.y, blockIdx.z != 0, gridDim.x, k, v, perm, Kt, Vt, kix, probe, by_index, listed, parts,
             tiles_per_block);
}
template <int D>
struct TileJob {
  TensorView k, v;
  const int32_t* perm;
  uint4 *Kt, *Vt;
  int tiles;
  __device__ __forceinline__ void run(int block) const {
    const int row = block / tiles, tile = block - row * tiles, heads = k.heads;
    const bool is_v = row >= heads;
    tile_kv<D>(tile, is_v ? row - heads : row, is_v, tiles, k, v, perm, Kt, Vt, nullptr, nullptr, 0, nullptr, 0, 1);
  }
};

// ---------------------------------------------------------------------------------
// Main kernel
// ---------------------------------------------------------------------------------
struct MfmaArgs {
  TensorView q; const char* Kt; const char* Vt;
  const int32_t* row_count; const int32_t* row_cols; int32_t cols_stride;
  const int32_t* perm_q;
  __bf16* out; float* lse;
  int Nq, Nk, Lq, Lk, group, wgs_per_head, total_wgs;
  float scale_log2e;
  int64_t out_sb, out_sh, out_sl;   // strides of out in elements
  int heads_q;
  const int32_t* kix;        // causal: [BHkv][tiles][kIxStride] original key indices of a tile, then their min and max
  int causal_off;            // causal: L_k - L_q
  const int32_t* probe;      // nullable: {blocks in the union of a group's lists, blocks in its lists} over sampled groups
  int run_if_solo;           // with probe: this launch runs iff (lists overlap little) == run_if_solo
  int32_t* redo;             // nullable, one word per workgroup: written by the pass without running maxima (1 = a row
                             // sum left the safe range), read by the pass with them, which skips workgroups at 0
  int stages;                // 512-query shape: tiles the LDS ring holds
  int splits;                // kSplit: workgroups that share a union list, and where they leave their rows:
  float* part_o;             //   [split][BHq][Lq][D] unnormalised, by sorted position
  float2* part_ml;           //   [split][BHq][Lq] running maximum (log2), running sum
};

// kGather: where the rows of the tiles are read from, in the order of perm_k (nullable).
struct RowSource {
  TensorView k, v;
  const int32_t* perm_k;
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

// The lane number made anew, opaque to the compiler, which would keep it (and what follows from it) in registers.
__device__ __forceinline__ int fresh_lane() {
  int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(l));
  return l;
}

// Per-wave state of the online softmax and the output accumulator.
template <int D>
struct WaveState {
  floatx16 o[Geo<D>::kDBlocks];
  float m_run, l_run;
  float lt;                  // kFast: the row sum of the half tile before this one
};

// max of three floats; this file is compiled with -fno-honor-nans (scores are finite or
// -inf), so no NaN canonicalisation is emitted and this becomes one v_max3_f32.
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// LDS byte address of a pointer into the workgroup's shared memory, and a 16-byte fragment read at one.
typedef const __attribute__((address_space(3))) char* lds_cptr_t;
typedef const __attribute__((address_space(3))) bf16x8* lds_frag_ptr_t;
__device__ __forceinline__ uint32_t lds_addr(const char* p) { return (uint32_t)(uintptr_t)(lds_cptr_t)p; }
__device__ __forceinline__ bf16x8 lds_frag(uint32_t addr) { return *(lds_frag_ptr_t)(uintptr_t)addr; }
typedef __attribute__((address_space(3))) short4v* lds_quad_ptr_t;
__device__ __forceinline__ bf16x4 lds_transposed(uint32_t addr) {
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad_ptr_t)(uintptr_t)addr));
}
__device__ const uint4 kZeroRow[16] = {};         // the row of a key that does not exist

// One 64-key tile: S^T, softmax, O^T update, reading the LDS stage at `stage`.  kMasked:
// keys at tile positions >= nvalid do not exist (ragged end of the sequence) and get -inf.
// kFast: no maximum is taken, the arithmetic of process_tile2's kFast form step by step (same bits).
// kGather: V as it stands in memory, one row of D values per key; vaddr0 is then row 4h + (lane / 4) % 4, chunk 2 (lane / 16 % 2) +
// lane % 4 / 2, half lane % 2 of it, where chunk c of row r sits at c ^ 4 (r & 3) (D = 64: c ^ 4 (r / 2 & 1)).
template <bool kMasked, int D, bool kFast, bool kGather>
__device__ __forceinline__ void process_tile(WaveState<D>& st, const bf16x8 (&qf)[Geo<D>::kKSteps], const char* stage,
                                             int kaddr0, int vaddr0, float c, int nvalid, int h) {
  const char* ks = stage;
  const char* vs = stage + Geo<D>::kTileBytes;
  // V^T of 16 keys (group g of the tile) and 32 dimensions: a lane's dimension, its eight keys in operand-slot order.  From rows
  // of V the transposing read gives lane i of 16 column i of the four rows that the 16 lanes address.
  auto vt_frag = [&](int g, int db) -> bf16x8 {
    if constexpr (kGather) {
      const uint32_t at = lds_addr(vs) + ((uint32_t)vaddr0 ^ (uint32_t)(db << 6)) + g * 16 * Geo<D>::kRowBytes;
      const bf16x4 lo = lds_transposed(at), hi = lds_transposed(at + 8 * Geo<D>::kRowBytes);
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      // chunk 2g+h of d-row li at position (2g+h) ^ ((li>>1)&7)
      return *reinterpret_cast<const bf16x8*>(vs + (vaddr0 ^ (g << 5)) + db * 32 * 128);
    }
  };

  // ---- S^T = K Q^T : two 32-key row blocks
  floatx16 s0 = {0}, s1 = {0};
#pragma unroll
  for (int s = 0; s < Geo<D>::kKSteps; ++s) {
    const int ka = kaddr0 ^ (s << 5);     // chunk 2s+h of row li at position (2s+h) ^ (li & (chunks per row - 1))
    const bf16x8 k0 = *reinterpret_cast<const bf16x8*>(ks + ka);
    const bf16x8 k1 = *reinterpret_cast<const bf16x8*>(ks + ka + 32 * Geo<D>::kRowBytes);
    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0, qf[s], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1, qf[s], s1, 0, 0, 0);
  }
  if (kMasked && nvalid < kTileKeys) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int kk = 8 * (r >> 2) + 4 * h + (r & 3);
      if (kk >= nvalid) s0[r] = -INFINITY;
      if (32 + kk >= nvalid) s1[r] = -INFINITY;
    }
  }
  if constexpr (kFast) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (__builtin_amdgcn_ballot_w64(st.lt > kSafeSum) != 0) {
        const float other = __shfl_xor(st.lt, 32);           // (by every lane, see process_tile2)
        const bool up = (st.lt > kSafeSum) | (other > kSafeSum);
        const float alpha = up ? kShiftMul : 1.f;
        st.m_run += up ? kShiftLog2 : 0.f;
        st.l_run *= alpha;
#pragma unroll
        for (int i = 0; i < Geo<D>::kDBlocks; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) st.o[i][r] *= alpha;
      }
      const floatx16& sh = half == 0 ? s0 : s1;
      bf16x8 pb[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) pb[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sh[r], c, -st.m_run));
      float la = 0.f;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 0, 1), ones, la, false);
        la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 2, 3), ones, la, false);
        la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 4, 5), ones, la, false);
        la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 6, 7), ones, la, false);
      }
      st.l_run += la;
      st.lt = la;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
#pragma unroll
        for (int db = 0; db < Geo<D>::kDBlocks; ++db) {
          const bf16x8 vv = vt_frag(2 * half + g, db);
          st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, pb[g], st.o[db], 0, 0, 0);
        }
      }
    }
    return;
  }
  // ---- online softmax in the log2 domain, lazy running max
  float mx = max3(s0[0], s1[0], s0[1]);
#pragma unroll
  for (int r = 1; r < 15; ++r) mx = max3(mx, s1[r], s0[r + 1]);
  mx = max3(mx, s1[15], __shfl_xor(max3(mx, s1[15], s1[15]), 32));
  const float mc = mx * c;
  if (__builtin_amdgcn_ballot_w64(mc > st.m_run + kLazyTau) != 0) {
    const float m_new = fmaxf(st.m_run, mc);
    const float alpha = __builtin_amdgcn_exp2f(st.m_run - m_new);
    st.m_run = m_new;
    st.l_run *= alpha;
#pragma unroll
    for (int i = 0; i < Geo<D>::kDBlocks; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.o[i][r] *= alpha;
  }
  const float m_use = st.m_run;
  bf16x8 pb[4];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    pb[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s0[r], c, -m_use));
    pb[2 + (r >> 3)][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s1[r], c, -m_use));
  }
  // row sum of the bf16-rounded probabilities (the values the second product consumes)
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  float lsum = st.l_run;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 0, 1), ones, lsum, false);
    lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 2, 3), ones, lsum, false);
    lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 4, 5), ones, lsum, false);
    lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 6, 7), ones, lsum, false);
  }
  st.l_run = lsum;

  // ---- O^T += V^T P^T
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int db = 0; db < Geo<D>::kDBlocks; ++db) {
      const bf16x8 vv = vt_frag(g, db);
      st.o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, pb[g], st.o[db], 0, 0, 0);
    }
  }
}

// Two query groups per wave (64 queries): the same arithmetic per query, but every K and V^T
// fragment read from LDS feeds two MFMAs (one per group), and the 64-key tile is walked as two
// 32-key halves so that only 32 score registers per group pair are live at a time.
template <int D>
struct WaveState2 {
  floatx16 o[2][Geo<D>::kDBlocks];
  float m_run[2], l_run[2];
  float lt[2];               // kFast: the row sums of the half tile before this one
};

// kQR of the k-steps take their Q^T fragments from registers; the others are read back from the
// wave's lane-private LDS area at `qs` ([group 2][k-step][lane] 16 bytes): O (128 registers) and all
// of Q (64) would leave the compiler too few of the 256 registers a wave has at two waves per SIMD.
// kCausal: kix4 points at the lane's four key indices of the tile's first group of eight keys
// (original positions, INT_MAX past the end of the sequence, which also covers the ragged tile); a
// key is visible to the query of group a / b iff its index does not exceed qla / qlb.
// kFast: no maximum is taken.  The reference m of a query only has to keep 2^(c s - m) inside the
// range of the formats (bf16 and fp32 share their exponent), it need not be the maximum: it starts at
// 0 and is raised by kShiftLog2 whenever the row sums of the half tile before, which are needed
// anyway, exceed kSafeSum.  The caller checks the final sums (kMinSum, kMaxSum) and has the rows
// computed again with running maxima if a sum has left the safe range.  Taking the maximum of every
// half tile (16 v_max3, two lane exchanges, and the wait of every exponential for the last score)
// was a quarter of the vector instructions of a tile.
template <bool kMasked, int D, int kQR, bool kCausal = false, bool kFast = false>
__device__ __forceinline__ void process_tile2(WaveState2<D>& st, const bf16x8 (&qa)[kQR], const bf16x8 (&qb)[kQR],
                                              const char* qs, const char* stage, int kaddr0, int vaddr0, float c,
                                              int nvalid, int h, const int* kix4 = nullptr, int qla = 0, int qlb = 0,
                                              int seen = 0) {
  constexpr int kQL = Geo<D>::kKSteps - kQR;               // k-steps whose Q^T fragments live in LDS
  // One LDS address per operand and tile; the k-step (group) is folded in by an xor at the point of
  // use (ring stages start at multiples of 32 KB, so the xor of bits 5-8 commutes with adding the
  // stage).  The two bases are opaque to the compiler, which would otherwise keep all twelve xor-ed
  // addresses in registers for the whole kernel and add the stage offset to each in every tile.
  uint32_t kbase = lds_addr(stage) + (uint32_t)kaddr0;
  uint32_t vbase = lds_addr(stage) + (uint32_t)(Geo<D>::kTileBytes + vaddr0);
  asm volatile("" : "+v"(kbase), "+v"(vbase));
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (kMasked && half == 1 && nvalid <= 32) break;        // wave-uniform: no key in the second half
    if (kCausal && half == 1 && (seen & 1)) break;          // wave-uniform: none that a query of the wave sees
    // the parked fragments are read again in every half: kept in registers across the halves they
    // would cost the 16 registers that parking them is meant to free
    asm volatile("" ::: "memory");
    floatx16 sa = {0}, sb = {0};
#pragma unroll
    for (int s = 0; s < Geo<D>::kKSteps; ++s) {
      const bf16x8 kf = lds_frag((kbase ^ (uint32_t)(s << 5)) + half * 32 * Geo<D>::kRowBytes);
      if (s < kQR) {
        sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qa[s < kQR ? s : 0], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qb[s < kQR ? s : 0], sb, 0, 0, 0);
      } else {
        const bf16x8 fa = *reinterpret_cast<const bf16x8*>(qs + (s - kQR) * 1024);
        const bf16x8 fb = *reinterpret_cast<const bf16x8*>(qs + (kQL + s - kQR) * 1024);
        sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, fa, sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, fb, sb, 0, 0, 0);
      }
    }
    if (!kCausal && kMasked && nvalid < kTileKeys) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int kk = 32 * half + 8 * (r >> 2) + 4 * h + (r & 3);
        if (kk >= nvalid) { sa[r] = -INFINITY; sb[r] = -INFINITY; }
      }
    }
    if (kCausal && !(seen & (2 << half))) {                 // wave-uniform: not every query sees all of the half
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int4 ix = *reinterpret_cast<const int4*>(kix4 + 32 * half + 8 * g4);
        const int ia[4] = {ix.x, ix.y, ix.z, ix.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (ia[e] > qla) sa[4 * g4 + e] = -INFINITY;
          if (ia[e] > qlb) sb[4 * g4 + e] = -INFINITY;
        }
      }
    }
    if constexpr (kFast) {
      if (__builtin_amdgcn_ballot_w64(st.lt[0] > kSafeSum || st.lt[1] > kSafeSum) != 0) {
        // a query's keys are split over two lanes (lane halves), which must move its reference together
        // (the exchanges first, by every lane: inside a short-circuit `||` only the lanes that still have
        //  to ask would be active, and a lane exchange reads 0 from an inactive lane)
        const float other_a = __shfl_xor(st.lt[0], 32), other_b = __shfl_xor(st.lt[1], 32);
        const bool ua = (st.lt[0] > kSafeSum) | (other_a > kSafeSum);
        const bool ub = (st.lt[1] > kSafeSum) | (other_b > kSafeSum);
        const float aa = ua ? kShiftMul : 1.f, ab = ub ? kShiftMul : 1.f;
        st.m_run[0] += ua ? kShiftLog2 : 0.f; st.m_run[1] += ub ? kShiftLog2 : 0.f;
        st.l_run[0] *= aa; st.l_run[1] *= ab;
#pragma unroll
        for (int i = 0; i < Geo<D>::kDBlocks; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) { st.o[0][i][r] *= aa; st.o[1][i][r] *= ab; }
      }
    } else {
      float mxa = max3(sa[0], sa[1], sa[2]), mxb = max3(sb[0], sb[1], sb[2]);
#pragma unroll
      for (int r = 3; r < 15; r += 2) { mxa = max3(mxa, sa[r], sa[r + 1]); mxb = max3(mxb, sb[r], sb[r + 1]); }
      mxa = fmaxf(mxa, sa[15]); mxb = fmaxf(mxb, sb[15]);
      // (exchanging the halves with v_permlane32_swap instead of the LDS permute measured 1 % slower)
      mxa = fmaxf(mxa, __shfl_xor(mxa, 32)); mxb = fmaxf(mxb, __shfl_xor(mxb, 32));
      const float mca = mxa * c, mcb = mxb * c;
      if (__builtin_amdgcn_ballot_w64(mca > st.m_run[0] + kLazyTau || mcb > st.m_run[1] + kLazyTau) != 0) {
        const float na = fmaxf(st.m_run[0], mca), nb = fmaxf(st.m_run[1], mcb);
        const float aa = __builtin_amdgcn_exp2f(st.m_run[0] - na), ab = __builtin_amdgcn_exp2f(st.m_run[1] - nb);
        st.m_run[0] = na; st.m_run[1] = nb;
        st.l_run[0] *= aa; st.l_run[1] *= ab;
#pragma unroll
        for (int i = 0; i < Geo<D>::kDBlocks; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) { st.o[0][i][r] *= aa; st.o[1][i][r] *= ab; }
      }
    }
    const float ma = st.m_run[0], mb = st.m_run[1];
    bf16x8 pa[2], pb[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      pa[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sa[r], c, -ma));
      pb[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sb[r], c, -mb));
    }
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float la = kFast ? 0.f : st.l_run[0], lb = kFast ? 0.f : st.l_run[1];
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pa[g], pa[g], 0, 1), ones, la, false);
      la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pa[g], pa[g], 2, 3), ones, la, false);
      la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pa[g], pa[g], 4, 5), ones, la, false);
      la = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pa[g], pa[g], 6, 7), ones, la, false);
      lb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 0, 1), ones, lb, false);
      lb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 2, 3), ones, lb, false);
      lb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 4, 5), ones, lb, false);
      lb = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pb[g], pb[g], 6, 7), ones, lb, false);
    }
    if constexpr (kFast) {
      st.l_run[0] += la; st.l_run[1] += lb;
      st.lt[0] = la; st.lt[1] = lb;
    } else {
      st.l_run[0] = la; st.l_run[1] = lb;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const uint32_t va = vbase ^ (uint32_t)((2 * half + g) << 5);
#pragma unroll
      for (int db = 0; db < Geo<D>::kDBlocks; ++db) {
        const bf16x8 vv = lds_frag(va + db * 32 * 128);
        st.o[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, pa[g], st.o[0][db], 0, 0, 0);
        st.o[1][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, pb[g], st.o[1][db], 0, 0, 0);
      }
    }
  }
}

// State of a wave by number of query groups, with uniform accessors for prologue and epilogue.
template <int D, int NG> struct StateOf { typedef WaveState<D> type; };
template <int D> struct StateOf<D, 2> { typedef WaveState2<D> type; };
template <int D>
__device__ __forceinline__ void init_state(WaveState<D>& st, bool fast = false) {
#pragma unroll
  for (int i = 0; i < Geo<D>::kDBlocks; ++i) st.o[i] = floatx16{0};
  st.m_run = fast ? 0.f : kNoMax;
  st.l_run = 0.f;
  st.lt = 0.f;
}
template <int D>
__device__ __forceinline__ void init_state(WaveState2<D>& st, bool fast = false) {
#pragma unroll
  for (int r = 0; r < 2; ++r) {
#pragma unroll
    for (int i = 0; i < Geo<D>::kDBlocks; ++i) st.o[r][i] = floatx16{0};
    st.m_run[r] = fast ? 0.f : kNoMax;
    st.l_run[r] = 0.f;
    st.lt[r] = 0.f;
  }
}
template <int D> __device__ __forceinline__ float l_of(const WaveState<D>& st, int) { return st.l_run; }
template <int D> __device__ __forceinline__ float m_of(const WaveState<D>& st, int) { return st.m_run; }
template <int D> __device__ __forceinline__ const floatx16& o_of(const WaveState<D>& st, int, int db) { return st.o[db]; }
template <int D> __device__ __forceinline__ float l_of(const WaveState2<D>& st, int r) { return st.l_run[r]; }
template <int D> __device__ __forceinline__ float m_of(const WaveState2<D>& st, int r) { return st.m_run[r]; }
template <int D> __device__ __forceinline__ const floatx16& o_of(const WaveState2<D>& st, int r, int db) { return st.o[r][db]; }

// kFast: has a final row sum left the range in which that pass is exact?  (On the bit patterns, which order like
// the values for positive floats and put inf, NaN and anything negative above kMaxSum: this file is compiled
// without NaN semantics for float comparisons.)
__device__ __forceinline__ bool sum_is_unsafe(float l) {
  return __float_as_uint(l) - __float_as_uint(kMinSum) > __float_as_uint(kMaxSum) - __float_as_uint(kMinSum);
}

__device__ __forceinline__ int64_t out_off(const MfmaArgs& a, int bhq, int row) {
  const int b = bhq / a.heads_q, hh = bhq - b * a.heads_q;
  return (int64_t)b * a.out_sb + (int64_t)hh * a.out_sh + (int64_t)row * a.out_sl;
}

// Dynamic LDS: [ring: stages x 32 KB][parked Q^T fragments][seq: Nk words][wave_counts: kWaves words].
// seq[i] = key block of the i-th entry of the union list | (bit 24+g set iff query block g of
// this workgroup lists it).  While seq is being built the ring area holds the per-key-block
// membership flags.
// kCausal (512-query shape only): the ring is followed by the original key indices of each stage's
// tile (with their bounds), scores are masked by original position, and a wave skips a tile or its second half if
// none of its keys is visible to any of the wave's queries, and the mask if all are to all.  With sorted sequences a
// block's indices are spread over the whole sequence; blocks of 128 are therefore walked by original index inside
// (tile_kv_kernel, positions_by_index): 32 heads, L = 32768, s = 0.5: 8579 us in perm's order, 7910 with hidden halves
// left out, 7209 without the masks that mask nothing.
// kSplit: a.splits workgroups share the query blocks and take equal runs of the union list each; their rows
// stay unnormalised and attn_combine_kernel adds them up.
// kGather (128-query shape): no tiles are laid out beforehand; the rows of K and V are fetched straight from the caller's
// tensors (the source address of a lane of a direct-to-LDS load is free), and V^T fragments come from rows of V.
// kPacked: among the jobs of a packed batch (that changes where the compiler puts the loop, see there).
template <int kB, int D, int kWgQueries, int kQPW, bool kCausal, bool kFast, bool kSplit, bool kGather = false, bool kPacked = false>
__device__ __forceinline__ void attn_mfma(const MfmaArgs& a, int logical, const RowSource* src = nullptr) {
  using G = Geo<D>;
  static_assert(!kCausal || (kQPW == 64 && kWgQueries == kWideQueries), "the causal path is built on the 512-query shape");
  static_assert(!kGather || (kQPW == 32 && kWgQueries == kSoloQueries), "rows are gathered by the 128-query shape");
  static_assert(!kFast || !kSplit, "the safe range of a row's sum is tested on the whole sum");
  static_assert(!kFast || (kQPW == 64 && kWgQueries == kWideQueries) || (kQPW == 32 && kWgQueries == kSoloQueries),
                "the pass without running maxima is built on the 512-query and the 128-query shape");
  // the 128-query shape has the registers to repeat itself with running maxima where that is needed; the
  // 512-query one leaves it to a second launch
  constexpr bool kRetry = kFast && kQPW == 32;
  constexpr int kWaves = kWgQueries / kQPW, kThreads = kWaves * 64, kQueriesPerWg = kWgQueries;
  constexpr int kNG = kQPW / 32;             // 32-query groups per wave: 1 or 2
  constexpr int kStages = stages_of(kThreads, kQPW);
  constexpr bool kSpans = kNG == 2 && wide_spans(D, kCausal, kFast);
  const int stages = kSpans ? a.stages : kStages;
  constexpr int kQR = q_reg_steps(D, kQPW, kCausal, kFast), kQL = G::kKSteps - kQR;
  constexpr int kQParkBytes = kWaves * kNG * kQL * 1024;
  constexpr int kTileBytes = G::kTileBytes, kStageBytes = G::kStageBytes;
  const int ring_bytes = stages * kStageBytes;
  constexpr int kLoadsPerWave = 2 * G::kChunksPerTile / kWaves;
  constexpr int NQB = kQueriesPerWg / kB;    // query blocks per workgroup: 2 or 4 (SOLO: 1 or 2)
  if (a.probe) {
    // the other shape of workgroup is launched too; exactly one of the two does the work.  A
    // 512-query workgroup walks the union of its 512 / B lists; four 128-query ones walk the
    // unions of their own 128 / B lists.  Measured break-even (wide 26.4 against 27.1 ms at a
    // ratio of 1.29, 157.7 against 143.6 ms at 1.64): the narrow shape wins once the wide union
    // exceeds about 1.35 times the average narrow one.
    const int uni = a.probe[0], uni_sub = a.probe[1];
    // At D = 64 a tile is half the bytes and the matrix work, and the narrow shape (half the registers, twice the
    // waves) hides its softmax better: level at ratios of 1.11 to 1.17 (2 % either way), ahead at 1.22 (1133 / 1003 us,
    // 32 heads, L = 32768; 3180 / 2895 us, 24 heads, L = 65536).
    constexpr int kBreakEven = D == 64 ? 119 : 135;
    const bool little_overlap = 100 * (int64_t)uni * 4 > kBreakEven * (int64_t)uni_sub;
    if ((int)little_overlap != a.run_if_solo) return;
  }
  constexpr int TPB = kB / kTileKeys;        // key tiles per key block: 2 or 1
  extern __shared__ __attribute__((aligned(16))) char smem[];
  uint32_t* flags = reinterpret_cast<uint32_t*>(smem);
  uint32_t* seq = reinterpret_cast<uint32_t*>(smem + ring_bytes + kQParkBytes);
  uint32_t* wave_counts = seq + a.Nk;
  int* kix_lds = reinterpret_cast<int*>(smem + ((ring_bytes + kQParkBytes + a.Nk * 4 + kWaves * 4 + 15) & ~15));   // kCausal

  int split = 0;
  if constexpr (kSplit) {
    split = logical % a.splits;
    logical /= a.splits;
  }
  // the pass with running maxima, launched behind the one without: only the workgroups that one gave up on
  if (!kFast && a.redo && a.redo[logical] == 0) return;
  const int bhq = logical / a.wgs_per_head, wg = logical - bhq * a.wgs_per_head;
  const int bhk = bhq / a.group;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 31, h = lane >> 5;
  const int grp = wave * kQPW / kB;                    // query block of this wave inside the wg
  const int nqb = min(NQB, a.Nq - wg * NQB);           // query blocks that exist
  // Sorted positions of the queries of thread t.  Causal with blocks of 128: the queries of a block are dealt to its
  // two waves by original index, the lower half to one and the upper half to the other (the order inside a block is
  // free), so that the wave of the lower half can leave out what lies beyond all its queries; of the two waves of
  // a SIMD, numbers w and w + 4, one has a lower and one an upper half.
  constexpr bool kByIndex = kCausal && kB == 128;
  auto positions_by_index = [&](int t, int (&pos)[2]) {
    int* raw = reinterpret_cast<int*>(smem);
    int* ordered = raw + kQueriesPerWg;
    const int p = wg * kQueriesPerWg + t, w = t >> 6;
    raw[t] = p < a.Lq ? perm_at(a.perm_q, (int64_t)bhq * a.Lq, p, a.Lq) : INT_MAX;
    __syncthreads();
    ordered[(t & ~127) + place_in_block(raw + (t & ~127), t & 127)] = p;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; ++r) pos[r] = ordered[(w >> 1) * 128 + ((w ^ (w >> 2)) & 1) * 64 + 32 * r + (t & 31)];
    __syncthreads();
  };
  const int pos0 = wg * kQueriesPerWg + wave * kQPW + li;   // sorted position of this lane's first query (next: +32)
  int qpos[2];                                              // kByIndex: of both
  if constexpr (kByIndex) positions_by_index(tid, qpos);
  auto position = [&](int r) -> int {
    if constexpr (kByIndex) return qpos[r];
    return pos0 + 32 * r;
  };

  // ---- union of the block lists of this workgroup's query blocks ------------------------
  // What the prologue reads by one address is requested before the first barrier, which waits for it: of every list (its
  // threads have one each) the count and the first entries, and the entry of perm_q.  One latency instead of two for each
  // list in turn and one for perm_q (attention call, both in one run): 8 heads, L = 2472, d = 64: 28.2 -> 27.6 us; 32 heads, L =
  // 16384, keep 10 %: 487 -> 480, 25 %: 1030 -> 1020; causal, blocks of 64, keep 50 %: 2209 -> 2190.  (With two query groups per
  // wave perm_q waits until the union is there: two entries kept across it change the compiler's registers for the whole
  // kernel: dense, L = 16384, 3494 against 3473; 32 heads, L = 131072, keep 50 %, 115.9 ms against 114.5; both in one run.)
  int q_raw = 0;
  if constexpr (kNG == 1) {
    const int pos = min(position(0), a.Lq - 1);
    q_raw = a.perm_q ? a.perm_q[(int64_t)bhq * a.Lq + pos] : pos;
  }
  constexpr int kPerList = kThreads / NQB;
  const int lg = tid / kPerList, l0 = tid % kPerList;
  const int64_t rowid = (int64_t)bhq * a.Nq + wg * NQB + min(lg, nqb - 1);
  const int32_t* cl = a.row_cols ? a.row_cols + rowid * a.cols_stride : nullptr;
  int l_count = 0, l_col = -1;
  if (a.row_cols) {
    l_count = a.row_count[rowid];
    l_col = cl[min(l0, a.cols_stride - 1)];
  }
  for (int c = tid; c < a.Nk; c += kThreads) flags[c] = a.row_cols ? 0u : ((1u << nqb) - 1u);
  __syncthreads();
  if (a.row_cols) {
    const int cnt = lg < nqb ? min(l_count, a.cols_stride) : 0;
    for (int i = l0; i < cnt; i += kPerList) {
      const int col = i == l0 ? l_col : cl[i];
      if ((unsigned)col < (unsigned)a.Nk) atomicOr(&flags[col], 1u << lg);     // anything else is ignored
    }
    __syncthreads();
  }
  // Q^T operand: lane (query li, half h) holds Q[q][16 s + 8 h .. +7] for s = 0..7
  bf16x8 qf[kNG][kQR];
  int q_lim[kNG];               // kCausal: the largest original key index the lane's query of each group may see
#pragma unroll
  for (int r = 0; r < kNG; ++r) q_lim[r] = INT_MIN;
  char* qpark = smem + ring_bytes + (wave * kNG * kQL) * 1024 + lane * 16;    // this lane's parked fragments
  auto load_q = [&]() {
#pragma unroll
    for (int r = 0; r < kNG; ++r) {
      // the query of sorted position qpos, read from the caller's tensor; positions past L_q
      // (padding of the last block, or a query block that does not exist) read row 0 and are never stored
      const int qpos = position(r);
      int qrow = 0;
      if (qpos < a.Lq) {
        if constexpr (kNG == 1) qrow = (unsigned)q_raw < (unsigned)a.Lq ? q_raw : qpos;          // (as perm_at)
        else qrow = perm_at(a.perm_q, (int64_t)bhq * a.Lq, qpos, a.Lq);
      }
      if (kCausal && qpos < a.Lq) q_lim[r] = qrow + a.causal_off;
      const uint4* qp = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a.q.ptr) +
                                                       (a.q.head_offset(bhq) + (int64_t)qrow * a.q.stride_l) * 2);
#pragma unroll
      for (int s = 0; s < G::kKSteps; ++s) {
        uint4 t = qp[2 * s + h];
        if (s < kQR) qf[r][s < kQR ? s : 0] = *reinterpret_cast<bf16x8*>(&t);
        else *reinterpret_cast<uint4*>(qpark + (r * kQL + s - kQR) * 1024) = t;    // read back by this lane only
      }
    }
  };
  // One query group per wave: requested here, the rows arrive while the union is built.  (Two groups: below; held
  // across the union they cost the register allocator its footing: 15 spills instead of 4, 10 % of the kernel.)
  if constexpr (kNG == 1) load_q();
  int n_union = 0;
  for (int base = 0; base < a.Nk; base += kThreads) {
    const int cidx = base + tid;
    const uint32_t f = cidx < a.Nk ? flags[cidx] : 0u;
    const uint64_t bal = __builtin_amdgcn_ballot_w64(f != 0u);
    if (lane == 0) wave_counts[wave] = __popcll(bal);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int cw = wave_counts[w];
      before += (w < wave) ? cw : 0;
      total += cw;
    }
    if (f != 0u) seq[n_union + before + __popcll(bal & ((1ull << lane) - 1ull))] = (uint32_t)cidx | (f << 24);
    n_union += total;
    __syncthreads();
  }
  // every thread has passed its last read of flags (the ring area) and seq is complete

  if constexpr (kSplit) {                    // this workgroup's run of the list
    const int u0 = n_union * split / a.splits;
    n_union = n_union * (split + 1) / a.splits - u0;
    seq += u0;
  }
  if (n_union == 0) {
    if constexpr (kSplit) {
      // nothing to add: a maximum of -inf and a sum of 0, whose row the combining pass does not read
      for (int r = 0; r < kNG; ++r) {
        const int pos = position(r);
        if (pos < a.Lq && h == 0)
          a.part_ml[((int64_t)split * (a.total_wgs / (a.splits * a.wgs_per_head)) + bhq) * a.Lq + pos] = make_float2(-INFINITY, 0.f);
      }
      return;
    }
    // no valid key block in any list of this workgroup (malformed input): its rows become zeros
    for (int r = 0; r < kNG; ++r) {
      const int pos = position(r);
      if (pos < a.Lq) {
        const int orow = perm_at(a.perm_q, (int64_t)bhq * a.Lq, pos, a.Lq);
        uint4* op = reinterpret_cast<uint4*>(a.out + out_off(a, bhq, orow));
        for (int i = 0; i < G::kChunksPerRow / 2; ++i) op[(G::kChunksPerRow / 2) * h + i] = make_uint4(0u, 0u, 0u, 0u);
        if (a.lse && h == 0) a.lse[(int64_t)bhq * a.Lq + orow] = -INFINITY;
      }
    }
    if (kFast && !kRetry && tid == 0) a.redo[logical] = 0;
    return;
  }
  int n_tiles = n_union * TPB;
  {
    // a ragged last key block may leave its trailing tile without any valid key
    const int last_col = (int)(seq[n_union - 1] & 0xffffffu);
    if (TPB == 2 && last_col * kB + kTileKeys >= a.Lk) n_tiles -= 1;
  }
  const int64_t tiles_per_head = (int64_t)a.Nk * TPB;
  const char* Kh = a.Kt + (int64_t)bhk * tiles_per_head * kTileBytes;
  const char* Vh = a.Vt + (int64_t)bhk * tiles_per_head * kTileBytes;

  // entry of union position i (wave-uniform value in an SGPR)
  auto entry_of = [&](int t) -> uint32_t {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)seq[t / TPB]);
  };
  // kGather: this lane's rows of a tile (those of its K chunks, and of its V chunks again), requested a tile ahead
  constexpr int kRowsPerLane = kLoadsPerWave / 2, kRowsPerLoad = 64 / G::kChunksPerRow;
  int rows[kGather ? kRowsPerLane : 1];
  auto pos_of = [&](int tile, int j) { return tile * kTileKeys + (j * kWaves + wave) * kRowsPerLoad + lane / G::kChunksPerRow; };
  auto request_rows = [&](int tile) {
    if constexpr (kGather) {
      if (src->perm_k) {
        const int32_t* pm = src->perm_k + (int64_t)bhk * a.Lk;
#pragma unroll
        for (int j = 0; j < kRowsPerLane; ++j) rows[j] = pm[(uint32_t)min(pos_of(tile, j), a.Lk - 1)];
      } else {
#pragma unroll
        for (int j = 0; j < kRowsPerLane; ++j) rows[j] = min(pos_of(tile, j), a.Lk - 1);
      }
    }
  };
  auto issue_rows = [&](int tile, int stage) {             // the rows of `tile` have been requested
    const char* kh = reinterpret_cast<const char*>(src->k.ptr) + src->k.head_offset(bhk) * 2;
    const char* vh = reinterpret_cast<const char*>(src->v.ptr) + src->v.head_offset(bhk) * 2;
    const uint32_t k_row = (uint32_t)src->k.stride_l * 2, v_row = (uint32_t)src->v.stride_l * 2;
    // (the places of a lane's chunks are the same in every tile and for every j)
    const int chunk = lane % G::kChunksPerRow, r = wave * kRowsPerLoad + lane / G::kChunksPerRow;
    const uint32_t kc = (uint32_t)(chunk ^ (r & (G::kChunksPerRow - 1))) * 16, vc = (uint32_t)(chunk ^ (D == 128 ? 4 * (r & 3) : 4 * (r >> 1 & 1))) * 16;
    char* dst = smem + stage * kStageBytes + wave * 1024;
    uint32_t at[kRowsPerLane];
#pragma unroll
    for (int j = 0; j < kRowsPerLane; ++j) {
      const int got = rows[kGather ? j : 0];
      at[j] = (unsigned)got < (unsigned)a.Lk ? got : min(pos_of(tile, j), a.Lk - 1);     // (as perm_at)
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(kh + (__umul24(at[j], k_row) + kc)), (lds_ptr_t)(dst + j * kWaves * 1024), 16, 0, 0);
    }
    if ((tile + 1) * kTileKeys <= a.Lk) {                  // uniform
#pragma unroll
      for (int j = 0; j < kRowsPerLane; ++j)
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)(vh + (__umul24(at[j], v_row) + vc)), (lds_ptr_t)(dst + kTileBytes + j * kWaves * 1024), 16, 0, 0);
    } else {
      // (keys that do not exist: their probability is 0, which an infinity would not survive)
#pragma unroll
      for (int j = 0; j < kRowsPerLane; ++j) {
        const char* from = pos_of(tile, j) < a.Lk ? vh + (__umul24(at[j], v_row) + vc) : reinterpret_cast<const char*>(kZeroRow);
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)from, (lds_ptr_t)(dst + kTileBytes + j * kWaves * 1024), 16, 0, 0);
      }
    }
  };
  // direct-to-LDS copy of tile `tile` into ring stage `stage`: 32 chunks of 1 KB, chunk
  // j*kWaves+wave by this wave (16 K chunks, then 16 V chunks)
  auto issue_tile = [&](int tile, int stage) {
    if constexpr (kGather) { issue_rows(tile, stage); return; }
    // (kept in registers the lane offset becomes three 64-bit addresses, and Q^T fragments go to scratch for them)
    const int lane_i = kSpans || kCausal ? fresh_lane() : lane;
    const char* kp = Kh + (int64_t)tile * kTileBytes;      // wave-uniform bases
    const char* vp = Vh + (int64_t)tile * kTileBytes;
#pragma unroll
    for (int j = 0; j < kLoadsPerWave; ++j) {
      const int cb = j * kWaves + wave;                   // wave-uniform: K chunks first, then V^T chunks
      const char* src = (cb < G::kChunksPerTile ? kp : vp) + (cb % G::kChunksPerTile) * 1024 + (uint32_t)(lane_i * 16);
      char* dst = smem + stage * kStageBytes + cb * 1024;
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)src, (lds_ptr_t)dst, 16, 0, 0);
    }
    if constexpr (kCausal) {
      // the tile's key indices, minimum and maximum: kIxStride ints = 17 lanes of 16 bytes
      if (wave == 0 && lane_i < kIxStride / 4) {
        const int32_t* src = a.kix + ((int64_t)bhk * tiles_per_head + tile) * kIxStride + lane_i * 4;
        __builtin_amdgcn_global_load_lds((gbl_ptr_t)src, (lds_ptr_t)(kix_lds + stage * kIxStride), 16, 0, 0);
      }
    }
  };
  auto tile_of = [&](int t) -> int {
    const int tt = min(t, n_tiles - 1);
    return (int)(entry_of(tt) & 0xffffffu) * TPB + (tt % TPB);
  };

  // prologue: the first tile (SHARED: the first pair; past the end: the last tile again, never read)
  auto issue_first = [&]() {
    request_rows(tile_of(0));
    issue_tile(tile_of(0), 0);
    request_rows(tile_of(1));
    if (kStages == 4) issue_tile(tile_of(1), 1);
  };
  issue_first();

  if constexpr (kNG == 2) load_q();
  // LDS byte offsets inside a stage.  K: row li (+32 for the second block), chunk 2s+h at
  // position (2s+h) ^ (li & 15).  V^T: d-row li (+32 db), chunk 2g+h at (2g+h) ^ ((li>>1)&7).
  // (step s / group g are folded in by xor with s<<5 / g<<5 at the point of use)
  const int kaddr = li * G::kRowBytes + ((h ^ (li & (G::kChunksPerRow - 1))) << 4);
  const int vquad = lane >> 2 & 3;
  const int vaddr = kGather ? (4 * h + vquad) * G::kRowBytes +
                                  (((2 * (lane >> 4 & 1) + (lane >> 1 & 1)) ^ (D == 128 ? 4 * vquad : 4 * (vquad >> 1))) << 4) + 8 * (lane & 1)
                            : li * 128 + ((h ^ ((li >> 1) & 7)) << 4);

  typename StateOf<D, kNG>::type st;
  init_state<D>(st, kFast);
  const float c = a.scale_log2e;
  // one 64-key tile of the ring, for the one or two query groups of this wave
  // causal: the largest limit among this wave's queries (lanes without a query ask for nothing); a tile
  // whose smallest key index lies beyond it has nothing for the wave, and neither has such a second half
  int wq_max = INT_MIN;
  if constexpr (kCausal) {
    wq_max = max(q_lim[0], q_lim[kNG - 1]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wq_max = max(wq_max, __shfl_xor(wq_max, off));
    wq_max = __builtin_amdgcn_readfirstlane(wq_max);
  }
  // ... and the smallest: a half whose largest index does not exceed it needs no mask
  int wq_min = INT_MAX;
  if constexpr (kCausal) {
    wq_min = min(q_lim[0] == INT_MIN ? INT_MAX : q_lim[0], q_lim[kNG - 1] == INT_MIN ? INT_MAX : q_lim[kNG - 1]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wq_min = min(wq_min, __shfl_xor(wq_min, off));
    wq_min = __builtin_amdgcn_readfirstlane(wq_min);
  }
  // bit 0: the second half has nothing for the wave; bits 1, 2: the first / second half needs no mask
  auto seen_of = [&](int stage_no) -> int {
    if constexpr (!kCausal) return 0;
    const int* bound = kix_lds + stage_no * kIxStride + kTileKeys;
    return (__builtin_amdgcn_readfirstlane(bound[1]) > wq_max ? 1 : 0) | (__builtin_amdgcn_readfirstlane(bound[2]) <= wq_min ? 2 : 0) |
           (__builtin_amdgcn_readfirstlane(bound[3]) <= wq_min ? 4 : 0);
  };
  auto tile = [&](auto masked, int stage_no, int nvalid, auto fast) {
    const char* stage = smem + stage_no * kStageBytes;
    if constexpr (kNG == 1) process_tile<decltype(masked)::value, D, decltype(fast)::value, kGather>(st, qf[0], stage, kaddr, vaddr, c, nvalid, h);
    else {
      // the lane half is needed by the masking code only (ragged tile, causal mask): taken from the
      // lane number there, it does not occupy a register through the main loop
      const int h2 = decltype(masked)::value || kCausal ? fresh_lane() >> 5 : 0;
      process_tile2<decltype(masked)::value, D, kQR, kCausal, kFast>(st, qf[0], qf[kNG - 1], qpark, stage, kaddr, vaddr, c, nvalid,
                                                                     h2, kix_lds + stage_no * kIxStride + 4 * h2, q_lim[0],
                                                                     q_lim[kNG - 1], seen_of(stage_no));
    }
  };
  int wk_min = INT_MAX;         // kCausal: the smallest original key index in the wave's own list
  auto tile_has_visible_keys = [&](int stage_no) -> bool {
    if constexpr (!kCausal) return true;
    const int kmin = __builtin_amdgcn_readfirstlane(kix_lds[stage_no * kIxStride + kTileKeys]);
    wk_min = min(wk_min, kmin);
    return kmin <= wq_max;
  };
  constexpr std::integral_constant<bool, kFast> kMode{};
  constexpr std::false_type kFull{};
  constexpr std::true_type kRagged{};
  const uint32_t my_bit = 1u << (24 + grp);

  // All tiles but the last: never ragged.  The last tile is peeled so that the masking code
  // (and its per-lane constants) stays out of the loop.  Loads are issued in tile order, so
  // "at most 2 tiles of my loads outstanding" means my part of tile t has landed; the barrier
  // then says everyone's part has, and that everyone is done with tile t-1, whose stage the
  // next load overwrites.
  // Tiles travel in PAIRS: ring stages {0,1} and {2,3} form two slots of two tiles, and the
  // workgroup meets at one barrier per pair (half as many barriers, half the skew cost).
  // Iteration p computes tiles 2p, 2p+1 from slot p%2 while tiles 2p+2, 2p+3 land in the other
  // slot; their loads are issued right after the barrier, which also says that every wave is
  // done with that other slot (pair p-1).  The union entries of later tiles are read from LDS
  // early and turned into scalars late, so their latency hides behind the arithmetic.
  if constexpr (kNG == 2 && !kSpans) {
    // 64 queries per wave: ONE call site for full tiles (a second inlined copy of the tile code
    // costs the register allocator its footing).  Tile t + 1 lands while tile t is computed.
    uint32_t e_cur = entry_of(0);
    int t = 0;
#pragma nounroll
    for (; t + 1 < n_tiles; ++t) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      issue_tile(tile_of(t + 1), (t + 1) & 1);
      const uint32_t raw_n = seq[(t + 1) / TPB];
      if ((e_cur & my_bit) && tile_has_visible_keys(t & 1)) tile(kFull, t & 1, kTileKeys, kMode);
      e_cur = (uint32_t)__builtin_amdgcn_readfirstlane((int)raw_n);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int nvalid = a.Lk - ((int)(e_cur & 0xffffffu) * TPB + (t % TPB)) * kTileKeys;
    if ((e_cur & my_bit) && tile_has_visible_keys(t & 1)) tile(kRagged, t & 1, nvalid, kMode);
  } else if constexpr (kNG == 2) {
    // The same in spans (wide_spans).  `win` holds, for the tiles lo, lo + 1, ... that have landed, one byte each: the
    // query blocks that list the tile and have yet to compute it.  Between two barriers every query block computes the
    // first of these tiles that is left to it; tile lo is then finished by all, and so are those after it that nobody
    // waits for, whose stages the next tiles take.  A block that does not list a tile works on a later one instead of
    // sitting it out, and computes its own tiles in the same order as before (same bits).  All waves work this out by
    // themselves in scalar registers, before the barrier: after it, or without barriers by progress words in LDS, the
    // chain of instructions and LDS round trips was exposed in every tile (3 to 6 % of the kernel).
    // Spans, in lists: 1.06 where the union is 1.135 (L = 131072, keep 50 %), 1.13 where it is 1.29 (L = 16384, 10 %).
    // Tile by tile -> spans: 32 heads, L = 131072: 119.5 -> 117.3 ms; L = 16384, keep 10 %: 667 -> 653 us (whole
    // operator); L = 32768, B = 64 (eight lists to a workgroup): 8350 -> 7960 us; dense: level.
    const uint32_t last = (uint32_t)n_tiles - 1, ring = (uint32_t)stages;
    auto wrap = [&](uint32_t i) { return i >= ring ? i - ring : i; };
    auto listed_by = [&](uint32_t e, uint32_t i) { return i < last ? e >> 24 : 0u; };      // (the last tile: below)
    auto entry_at = [&](uint32_t i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)seq[min(i, last) / (uint32_t)TPB]); };
    uint32_t lo = 0, issued = 1, slot = 0, issue_slot = 1, stage_no = 0;
    uint32_t e0 = entry_at(1), e1 = entry_at(2);       // of the next two tiles to request
    uint32_t win = listed_by(entry_at(0), 0), mine = win >> grp & 0x01010101u;
    // Where the loop starts in a line of 64 bytes: at 56, blocks of 64 at 20.  What the compiler puts between this and the loop (some 400
    // bytes) decides how many instructions that takes; a test reads the offsets of the four forms from the code object, and fails where
    // that has moved them.  At 56 / 0 / 20 / 36, in turn on one card, three times: blocks of 128: dense, L = 16384: 3586 / 3595 / 3623 / 3619
    // us, 128K, keep 50 %: 117.8 / 118.0 / 118.7 / 118.7 ms, video 75K: 25845 / 25936 / 26113 / 26085 us, a packed batch of six: 721 / 722 / 726 /
    // 726; of 64: 32 heads, L = 50000, keep 25 %: 10902 / 10891 / 10815 / 10832, L = 32768: 8205 / 8186 / 8126 / 8165, the batch: 737 / 737 / 733 / 733.
    constexpr int kNops = (kB == 128 ? 2 : 9) - (kPacked ? 1 : 0);
    asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"n"(kNops));
#pragma nounroll
    while (lo < last || issued <= last) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const uint32_t here = issued - lo, want = min(min(last + 1 - issued, ring - here), 2u);
      if (want > 0) issue_tile((int)((e0 & 0xffffffu) * TPB + issued % TPB), (int)issue_slot);
      if (want > 1) issue_tile((int)((e1 & 0xffffffu) * TPB + (issued + 1) % TPB), (int)wrap(issue_slot + 1));
      if (mine != 0u && tile_has_visible_keys((int)stage_no)) tile(kFull, (int)stage_no, kTileKeys, kMode);
      // what the next span does
      uint32_t before = win | win << 8;                // byte j: who had one of the tiles 0 .. j to do
      before |= before << 16;
      const uint32_t rest = win & before << 8;
      const uint32_t done = rest ? (uint32_t)__builtin_ctz(rest) >> 3 : min(here, last - lo);
      const uint32_t fresh = (want > 0 ? listed_by(e0, issued) : 0u) | (want > 1 ? listed_by(e1, issued + 1) << 8 : 0u);
      win = (uint32_t)((rest | (uint64_t)fresh << 8 * here) >> 8 * done);
      lo += done;
      slot = wrap(slot + done);
      issued += want;
      issue_slot = wrap(issue_slot + want);
      mine = win >> grp & 0x01010101u;
      stage_no = wrap(slot + (mine ? (uint32_t)__builtin_ctz(mine) >> 3 : 0u));
      e0 = entry_at(issued);
      e1 = entry_at(issued + 1);
    }
    // the last tile, which may be ragged: the masks stay out of the loop
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const uint32_t e_last = entry_of(n_tiles - 1);
    const int nvalid = a.Lk - ((int)(e_last & 0xffffffu) * TPB + ((n_tiles - 1) % TPB)) * kTileKeys;
    const int last_stage = (int)(issue_slot == 0 ? ring - 1 : issue_slot - 1);
    if ((e_last & my_bit) && tile_has_visible_keys(last_stage)) tile(kRagged, last_stage, nvalid, kMode);
  } else if constexpr (kStages == 4) {
  uint32_t e_a = entry_of(0);
  uint32_t e_b = entry_of(min(1, n_tiles - 1));
  int t = 0;
  for (; t + 2 < n_tiles; t += 2) {          // pairs that do not contain the last tile
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int tf0 = min(t + 2, n_tiles - 1), tf1 = min(t + 3, n_tiles - 1);
    const uint32_t raw_f0 = seq[tf0 / TPB], raw_f1 = seq[tf1 / TPB];
    const int slot_next = ((t >> 1) + 1) & 1;
    {
      const int b0 = __builtin_amdgcn_readfirstlane((int)raw_f0) & 0xffffff;
      const int b1 = __builtin_amdgcn_readfirstlane((int)raw_f1) & 0xffffff;
      issue_tile(b0 * TPB + (tf0 % TPB), 2 * slot_next);
      issue_tile(b1 * TPB + (tf1 % TPB), 2 * slot_next + 1);
    }
    const int slot = ((t >> 1) & 1) * 2;            // first ring stage of the pair
    if (e_a & my_bit) tile(kFull, slot, kTileKeys, kMode);
    if (e_b & my_bit) tile(kFull, slot + 1, kTileKeys, kMode);
    e_a = (uint32_t)__builtin_amdgcn_readfirstlane((int)raw_f0);
    e_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)raw_f1);
  }
  {
    // the last pair: one or two tiles, the very last one possibly ragged
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int slot = ((t >> 1) & 1) * 2;
    if (t + 1 < n_tiles) {
      if (e_a & my_bit) tile(kFull, slot, kTileKeys, kMode);
      const int nvalid = a.Lk - ((int)(e_b & 0xffffffu) * TPB + ((t + 1) % TPB)) * kTileKeys;
      if (e_b & my_bit) tile(kRagged, slot + 1, nvalid, kMode);
    } else {
      const int nvalid = a.Lk - ((int)(e_a & 0xffffffu) * TPB + (t % TPB)) * kTileKeys;
      if (e_a & my_bit) tile(kRagged, slot, nvalid, kMode);
    }
  }
  } else {
    // SOLO: two stages, one tile per barrier; tile t+1 lands while tile t is computed
    auto walk = [&](auto fast) {
      uint32_t e_cur = entry_of(0);
      int t = 0;
      for (; t + 1 < n_tiles; ++t) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const uint32_t raw_n = seq[(t + 1) / TPB];
        const uint32_t e_nxt = (uint32_t)__builtin_amdgcn_readfirstlane((int)raw_n);
        issue_tile((int)(e_nxt & 0xffffffu) * TPB + ((t + 1) % TPB), (t + 1) & 1);
        request_rows(tile_of(t + 2));
        if (e_cur & my_bit) tile(kFull, t & 1, kTileKeys, fast);
        e_cur = e_nxt;
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const int nvalid = a.Lk - ((int)(e_cur & 0xffffffu) * TPB + (t % TPB)) * kTileKeys;
      if (e_cur & my_bit) tile(kRagged, t & 1, nvalid, fast);
    };
    walk(kMode);
    if constexpr (kRetry) {
      const float l_all = l_of(st, 0) + __shfl_xor(l_of(st, 0), 32);
      // (the barrier inside also says that every wave is done with the ring)
      if (__syncthreads_or(pos0 < a.Lq && sum_is_unsafe(l_all))) {
        init_state<D>(st, false);
        issue_first();
        walk(std::false_type{});
      }
    }
  }

  // ---- epilogue: normalise, scatter rows to their original positions
  // positions and lane halves are rebuilt from the thread index (opaque to the compiler): carried
  // through the main loop they would take registers that the accumulators and Q^T fragments need
  int tid_e = threadIdx.x;
  asm volatile("" : "+v"(tid_e));
  const int h_e = (tid_e >> 5) & 1;
  const int pos_e = wg * kQueriesPerWg + (tid_e >> 6) * kQPW + (tid_e & 31);
  int qpos_e[2];
  // Whether some row's sum left the safe range is settled before the rows are stored: the vote waits for all that the
  // workgroup has in flight, and behind the stores that was their way to memory, with every compute unit writing at once.
  if constexpr (kFast && !kRetry) {
    int unsafe = 0;
#pragma unroll
    for (int r = 0; r < kNG; ++r) {
      const float l_part = l_of(st, r), l_tot = l_part + __shfl_xor(l_part, 32);
      // (causal: a query that sees no key of its list has the sum 0 and is done; there are one or two such queries
      //  per head, and repeating their workgroups took 1210 us after the 8579 of this pass at 32 heads, L = 32768)
      if ((kCausal ? q_lim[r] >= wk_min : pos_e + 32 * r < a.Lq) && sum_is_unsafe(l_tot)) unsafe = 1;
    }
    const int any = __syncthreads_or(unsafe);
    if (tid_e == 0) a.redo[logical] = any;
  } else {
    __syncthreads();
  }                                            // (the ring, which others may still read, is used below)
  if constexpr (kByIndex) positions_by_index(tid_e, qpos_e);
  // A lane holds four neighbouring dimensions of its query at a time: stored from there, an instruction touches 32 rows for 16
  // bytes each (10.4 us of a workgroup's 125 at 32 heads, L = 16384, keep 10 %).  The rows of a group of queries therefore go through
  // LDS, in the wave's own part of the ring (chunk c of row r at c ^ (r & (chunks per row - 1))), and are written as whole rows.
  const int wave_e = __builtin_amdgcn_readfirstlane(tid_e >> 6), lane_e = tid_e & 63;
  char* const area = smem + wave_e * 32 * G::kRowBytes;
  char* const mine_e = area + (lane_e & 31) * G::kRowBytes;
  const int swz_e = lane_e & (G::kChunksPerRow - 1);
  constexpr int kRowsPerStore = 64 / G::kChunksPerRow;
  const int sub_e = lane_e % G::kChunksPerRow, row_e = lane_e / G::kChunksPerRow;
#pragma unroll
  for (int r = 0; r < kNG; ++r) {
    float l_part = l_of(st, r);
    const float m_fin = m_of(st, r);
    asm volatile("" : "+v"(l_part));             // (its exchange stays behind the barrier, which would have to wait for it)
    const float l_tot = l_part + __shfl_xor(l_part, 32);
    const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;    // a query block without any valid key block: zeros
    int pos = pos_e + 32 * r;
    if constexpr (kByIndex) pos = qpos_e[r];
    const int h = h_e;
    if constexpr (kSplit) {
      const int64_t row0 = ((int64_t)split * (a.total_wgs / (a.splits * a.wgs_per_head)) + bhq) * a.Lq;
      const int to = pos < a.Lq ? pos : -1;
      if (to >= 0 && h == 0) a.part_ml[row0 + pos] = make_float2(m_fin, l_tot);
      // (fp32: half a row at a time)
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int db = 0; db < G::kDBlocks / 2; ++db)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            floatx4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = o_of(st, r, half * (G::kDBlocks / 2) + db)[4 * r4 + e];
            *reinterpret_cast<floatx4*>(mine_e + (((8 * db + 2 * r4 + h) ^ swz_e) << 4)) = t;
          }
#pragma unroll
        for (int i = 0; i < 32 / kRowsPerStore; ++i) {
          const int row = i * kRowsPerStore + row_e, at = __shfl(to, row);
          const floatx4 t = *reinterpret_cast<const floatx4*>(area + row * G::kRowBytes + ((sub_e ^ (row & (G::kChunksPerRow - 1))) << 4));
          if (at >= 0) *reinterpret_cast<floatx4*>(a.part_o + (row0 + at) * D + half * (D / 2) + 4 * sub_e) = t;
        }
      }
    } else {
      const int orow = pos < a.Lq ? perm_at(a.perm_q, (int64_t)bhq * a.Lq, pos, a.Lq) : -1;
#pragma unroll
      for (int db = 0; db < G::kDBlocks; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          bf16x4 pk;
#pragma unroll
          for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o_of(st, r, db)[4 * r4 + e] * inv_l);
          *reinterpret_cast<bf16x4*>(mine_e + (((4 * db + r4) ^ swz_e) << 4) + 8 * h) = pk;
        }
      __bf16* const out_head = a.out + out_off(a, bhq, 0);
#pragma unroll
      for (int i = 0; i < 32 / kRowsPerStore; ++i) {
        const int row = i * kRowsPerStore + row_e, at = __shfl(orow, row);
        const bf16x8 t = *reinterpret_cast<const bf16x8*>(area + row * G::kRowBytes + ((sub_e ^ (row & (G::kChunksPerRow - 1))) << 4));
        if (at >= 0) *reinterpret_cast<bf16x8*>(out_head + (int64_t)at * a.out_sl + 8 * sub_e) = t;
      }
      if (a.lse && h == 0 && orow >= 0)
        a.lse[(int64_t)bhq * a.Lq + orow] = (m_fin + __log2f(l_tot)) * 0.6931471805599453f;
    }
  }
}

// XCD-aware order: consecutive workgroup ids go round-robin over the 8 XCDs; give each
// XCD a contiguous range of (head, query blocks) so that its L2 sees one head at a time.
__device__ __forceinline__ int xcd_order(int total) {
  return (total & 7) == 0 ? (blockIdx.x & 7) * (total >> 3) + (blockIdx.x >> 3) : blockIdx.x;
}
template <int kB, int D, int kWgQueries, int kQPW, bool kCausal = false, bool kFast = false, bool kSplit = false>
__global__ __launch_bounds__(kWgQueries / kQPW * 64, kWgQueries / kQPW == 8 ? 1 : 2) void attn_mfma_kernel(MfmaArgs a) {
  attn_mfma<kB, D, kWgQueries, kQPW, kCausal, kFast, kSplit>(a, xcd_order(a.total_wgs));
}
template <int kB, int D, bool kFast, bool kSplit>
__global__ __launch_bounds__(kSoloQueries / 32 * 64, 2) void attn_rows_kernel(MfmaArgs a, RowSource src) {
  attn_mfma<kB, D, kSoloQueries, 32, false, kFast, kSplit, true>(a, xcd_order(a.total_wgs), &src);
}
template <int kB, int D>
struct AttnJob {
  MfmaArgs a;
  __device__ __forceinline__ void run(int block) const { attn_mfma<kB, D, kSoloQueries, 32, false, true, false, false, true>(a, block); }
};
// The 512-query shape: the pass without running maxima, and the one with them for what that gave up on.
template <int kB, int D, bool kFast>
struct WideJob {
  MfmaArgs a;
  __device__ __forceinline__ void run(int block) const { attn_mfma<kB, D, kWideQueries, 64, false, kFast, false, false, true>(a, block); }
};

size_t sz_kv(int BHkv, int Nk, int B, int d) { return align_up((size_t)BHkv * Nk * B * d * 2, 256); }
size_t sz_kix(int BHkv, int Nk, int B) { return align_up((size_t)BHkv * (Nk * B / kTileKeys) * kIxStride * 4, 256); }

// Do the bitmaps of the listed blocks cost less than the tiles they save?  They take 5 us and 5 us per million list
// entries (the atomics of a row meet in the same words); the tiles move kv_bytes four times at 5.6 TB/s, and with lists
// of a share f of the blocks about (1 - f)^1.5 / 2 of that time is saved: rows of a KV head add up to much more than one
// of them.  Tiling, all blocks -> listed ones by the bitmaps: 32 heads, L = 16384, keep 10 / 25 / 50 %: 90 -> 32, 87 -> 46,
// 85 -> 68 us; 32 heads, 256 queries of 32768, 25 %: 188 -> 55; 32 heads on 8, L = 100000, B = 64 (6252 rows per KV head), 10 %:
// 139 -> 105; against, same sizes, 25 / 50 / 75 %: 138 -> 188, 137 -> 313, 137 -> 428; 8 heads, L = 24000, B = 64, 50 %: 35 -> 40.
bool bitmaps_pay(size_t kv_bytes, double f, double entries) {
  const double tiling_us = 4.0 * (double)kv_bytes / 5.6e6;
  return tiling_us * 0.5 * (1.0 - f) * std::sqrt(1.0 - f) > 5.0 + 5e-6 * entries;
}
size_t sz_listed(int BHkv, int Nk) { return align_up((size_t)BHkv * kListedParts * ceil_div(Nk, 32) * 4, 256); }

template <int kB, int D, int kWgQueries, int kQPW, bool kCausal, bool kFast, bool kSplit>
basa_status launch_main(MfmaArgs m, int BHq, hipStream_t st) {
  constexpr int kThreads = kWgQueries / kQPW * 64;
  m.stages = launch_stages<D>(kThreads, kQPW, m.Nk, kCausal, kFast);
  const size_t lds = lds_bytes<D>(kThreads, kQPW, m.Nk, kCausal, kFast, m.stages);
  // while the union list is built, the per-key-block membership flags live in the ring area
  if ((size_t)m.Nk * 4 > (size_t)stages_of(kThreads, kQPW) * Geo<D>::kStageBytes) {
    set_error("attention: %d key blocks exceed the %zu this workgroup shape can list", m.Nk,
              (size_t)stages_of(kThreads, kQPW) * Geo<D>::kStageBytes / 4);
    return BASA_ERR_UNSUPPORTED;
  }
  m.wgs_per_head = ceil_div(m.Nq * kB, kWgQueries);
  m.total_wgs = BHq * m.wgs_per_head * (kSplit ? m.splits : 1);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_mfma_kernel<kB, D, kWgQueries, kQPW, kCausal, kFast, kSplit>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");
  hipLaunchKernelGGL((attn_mfma_kernel<kB, D, kWgQueries, kQPW, kCausal, kFast, kSplit>), dim3(m.total_wgs), dim3(kThreads), lds, st, m);
  BASA_HIP_CHECK_LAUNCH("attn_mfma_kernel");
  return BASA_OK;
}
// dispatch on block size and head dimension
template <int kWgQueries, int kQPW, bool kCausal = false, bool kFast = false, bool kSplit = false>
basa_status launch_shape(const MfmaArgs& m, int B, int d, int BHq, hipStream_t st) {
  if (d == 128) return B == 128 ? launch_main<128, 128, kWgQueries, kQPW, kCausal, kFast, kSplit>(m, BHq, st)
                                : launch_main<64, 128, kWgQueries, kQPW, kCausal, kFast, kSplit>(m, BHq, st);
  return B == 128 ? launch_main<128, 64, kWgQueries, kQPW, kCausal, kFast, kSplit>(m, BHq, st)
                  : launch_main<64, 64, kWgQueries, kQPW, kCausal, kFast, kSplit>(m, BHq, st);
}
// The 128-query shape on rows of K and V (whole lists without running maxima, or split ones).
template <int kB, int D, bool kFast, bool kSplit>
basa_status launch_rows_of(MfmaArgs m, const RowSource& src, int BHq, hipStream_t st) {
  m.wgs_per_head = ceil_div(m.Nq * kB, kSoloQueries);
  m.total_wgs = BHq * m.wgs_per_head * (kSplit ? m.splits : 1);
  const size_t lds = lds_bytes<D>(kSoloQueries * 2, 32, m.Nk, false, kFast);
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_rows_kernel<kB, D, kFast, kSplit>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");
  hipLaunchKernelGGL((attn_rows_kernel<kB, D, kFast, kSplit>), dim3(m.total_wgs), dim3(kSoloQueries * 2), lds, st, m, src);
  BASA_HIP_CHECK_LAUNCH("attn_rows_kernel");
  return BASA_OK;
}
template <bool kFast, bool kSplit>
basa_status launch_rows(const MfmaArgs& m, const RowSource& src, int B, int d, int BHq, hipStream_t st) {
  if (d == 128) return B == 128 ? launch_rows_of<128, 128, kFast, kSplit>(m, src, BHq, st) : launch_rows_of<64, 128, kFast, kSplit>(m, src, BHq, st);
  return B == 128 ? launch_rows_of<128, 64, kFast, kSplit>(m, src, BHq, st) : launch_rows_of<64, 64, kFast, kSplit>(m, src, BHq, st);
}
// The 512-query shape in two passes: without running maxima, then, for the workgroups whose row sums
// left the safe range (none on ordinary inputs: that launch returns at once), with them.
template <bool kCausal>
basa_status launch_wide(MfmaArgs m, int B, int d, int BHq, int32_t* redo, bool two_pass, hipStream_t st) {
  if (two_pass) {
    m.redo = redo;
    const basa_status s = launch_shape<kWideQueries, 64, kCausal, true>(m, B, d, BHq, st);
    if (s != BASA_OK) return s;
  } else {
    m.redo = nullptr;
  }
  return launch_shape<kWideQueries, 64, kCausal, false>(m, B, d, BHq, st);
}

// Calls whose workgroups do not fill the device (fewer than two of 512 queries per compute unit, `small`): the shape
// (512 or 128 queries per workgroup) and the number of workgroups that share a list, from an estimate of the
// time.  Lists are split on the 128-query shape (split 512-query workgroups measure no better: 75 against 72 us,
// dense, 8 heads, L = 4100, d = 64), on the 512-query one only for the causal kernel, which has no
// other.
// One step of a 64-key tile, measured at D = 128: 2.95 us for a workgroup of 512 queries (causal: 3.4), 1.95 us for
// two of 128 that share a compute unit, 1.25 us for one alone; 0.63 of that at D = 64; 20 us of prologue and epilogue per
// round of workgroups of 512 queries (25 us of lists of one block, where nothing overlaps them), 10 us of 128, 4 us for the
// combining pass, and the partial rows at 2 TB/s written and read.  (From before the epilogue wrote whole rows, 5 us less for 512
// queries, and before the combining pass requested its parts together.)
// Attention call (tiling of K and V included), one workgroup of 512 queries per list -> this rule:
// 256 queries against 32K keys, 32 heads on 8, keep 25 %: 351 -> 98 us (128 queries, 8 workgroups per list);
// 8 heads, L = 2472, d = 64: 63 -> 28 us; 16 heads, L = 1977: 81 -> 36 us; dense, 8 heads, L = 12000, d = 128: 560 us,
// unchanged (the 128-query shape would take 624).
// Lists of up to 32 tiles stay whole, and a whole list on the 128-query shape gives the same bits as on the 512-query one.  Splitting
// them did not pay with the combining pass of the time (16 heads, L = 1977, 16 tiles: 39 us whole, 47 in two; 8 heads, L =
// 2472, d = 64, 20 tiles: 31 and 36; not so the causal kernel, 8 heads, L = 2100: 94 and 59 in six).  With the present one it does
// where few workgroups are there (whole / split, keep 50 %, d = 128: 1 head, L = 2472: 31.0 / 18.9, 4: 31.2 / 29.3, 8: level; 8 heads, 300
// queries of 4000: 46.4 / 20.8; 1 head, L = 600, d = 64: 12.5 / 13.4): this line is older than that.
constexpr int kCUs = 256, kMaxSplits = 32, kMinSplitTiles = 32;
constexpr double kWideStepUs = 2.95, kCausalStepUs = 3.4, kSoloPairStepUs = 1.95, kSoloStepUs = 1.25;
constexpr double kWideRoundUs = 20.0, kCausalRoundUs = 8.0, kSoloRoundUs = 10.0;
constexpr double step_scale(int d) { return d == 128 ? 1.0 : 0.63; }
// Blocks in the union of two lists of 64 queries and of the lists of 512, over one list, for lists that leave out `dead` of all.
constexpr double union_of_pair(int B, double dead) { return 1.0 + (B == 64 ? 0.1 : 0.0) * dead; }
constexpr double union_of_groups(int groups, double dead) { return 1.0 + 0.1 * (groups - 1) * dead; }
struct Plan { bool solo; int splits; double us; };
// Up to six of 512 queries per compute unit, whole lists only: there a last round that is mostly empty decides, and the
// 128-query shape has to be 5 % ahead by the estimate.  512-query -> chosen shape: 16 heads, L = 20000, keep 10 %
// (2.5 rounds): 388 -> 338 us; 24 heads, L = 12500, B = 64, keep 25 %: 644 -> 547; 32 heads, L = 9000, B = d = 64, keep
// 10 %: 145 -> 104; kept at 512 queries: 32 heads, L = 16384, keep 10 % (four full rounds, 461 either way).
constexpr int kSmallRounds = 2, kPlannedRounds = 6;
Plan plan_call(int BHq, int Nq, int Nk, int Lq, int B, int d, int list_len, bool causal, bool small, size_t part_bytes) {
  const size_t row_bytes = (size_t)BHq * Lq * (d * 4 + 8);
  const double dead = 1.0 - (double)list_len / Nk, scale = step_scale(d);
  Plan best{false, 1, 0.0};
  for (int solo = 0; solo <= (causal ? 0 : 1); ++solo) {
    const int queries = solo ? kSoloQueries : kWideQueries;
    const int64_t wgs = (int64_t)BHq * ceil_div(Nq * B, queries);
    // blocks in the union of a workgroup's lists, measured (full method): the union over 512 queries is 1.14 times that
    // over 128 at 50 %, 1.22 at 75 %, 1.29 at 90 %; two lists of 64 queries make about 1.05 to 1.1
    const int groups = solo ? 1 : std::min(4, ceil_div(Nq * B, kSoloQueries));
    const double uni = std::min((double)Nk, list_len * (Nq > 1 ? union_of_pair(B, dead) : 1.0) * union_of_groups(groups, dead));
    const bool may_split = small && (solo != 0) != causal && (causal || list_len * (B / kTileKeys) > kMinSplitTiles);
    for (int s = 1; s == 1 || (may_split && s <= kMaxSplits && uni >= s && s * row_bytes <= part_bytes); ++s) {
      const int64_t per_cu = (wgs * s + kCUs - 1) / kCUs;
      const double rounds = solo ? (double)((per_cu + 1) / 2) : (double)per_cu;
      const double step_us = solo ? (double)(per_cu / 2) * kSoloPairStepUs + (double)(per_cu % 2) * kSoloStepUs
                                  : (double)per_cu * (causal ? kCausalStepUs : kWideStepUs);
      const double round_us = solo ? kSoloRoundUs : causal ? kCausalRoundUs : kWideRoundUs;
      const double cost = std::ceil(uni / s) * (B / kTileKeys) * step_us * scale + round_us * rounds +
                          (s > 1 ? 4.0 + (double)(s * row_bytes) / 2e6 : 0.0);
      if ((!solo && s == 1) || cost < best.us * (small ? 1.0 : 0.95)) best = Plan{solo != 0, s, cost};
    }
  }
  return best;
}
// Room for the partial rows of as many workgroups per list as could be of use: two rounds of workgroups.
size_t part_bytes_of(int BHq, int Lq, int Nk, int B, int d, bool causal) {
  if (!causal && Nk * (B / kTileKeys) <= kMinSplitTiles) return 0;
  const int64_t splits = std::min<int64_t>(std::min(kMaxSplits, Nk), 8 * kCUs / ((int64_t)BHq * ceil_div(Lq, kSoloQueries)));
  return splits < 2 ? 0 : (size_t)splits * BHq * Lq * (d * 4 + 8);
}

// How much the lists of the query blocks that would share a 512-query workgroup have in common, on
// every kProbeStride-th such group of gsz = 512 / B neighbouring blocks: probe[0] += blocks in the
// union of the group's lists (what a 512-query workgroup walks), probe[1] += the same for each of
// the group's four 128-query subgroups, added up (what four 128-query workgroups walk; for B = 128
// simply the blocks in the four lists).  One wave per group: the lists are or-ed into bitmaps in LDS.
constexpr int kProbeStride = 8, kProbeMaxBlocks = 8192;
__global__ __launch_bounds__(256) void list_overlap_kernel(const int32_t* __restrict__ row_count,
                                                           const int32_t* __restrict__ row_cols, int cols_stride,
                                                           int Nq, int Nk, int gsz, int groups_total,
                                                           int32_t* __restrict__ probe) {
  __shared__ uint32_t bits[4][kProbeMaxBlocks / 32], sub[4][kProbeMaxBlocks / 32];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int group = (blockIdx.x * 4 + wv) * kProbeStride;
  const bool active = group < groups_total;             // no early exit: every wave meets the barriers
  const int groups_per_head = Nq / gsz;
  const int bh = active ? group / groups_per_head : 0, g0 = active ? (group - bh * groups_per_head) * gsz : 0;
  const unsigned limit = (unsigned)min(Nk, kProbeMaxBlocks);
  const int words = (int)((limit + 31) >> 5);
  const int rows_per_sub = gsz / 4;                     // query blocks of a 128-query subgroup: 1 or 2
  for (int w = lane; w < words; w += 64) bits[wv][w] = 0u;
  int uni_sub = 0;
  for (int sg = 0; sg < 4; ++sg) {
    for (int w = lane; w < words; w += 64) sub[wv][w] = 0u;
    __syncthreads();
    for (int r = 0; r < rows_per_sub; ++r) {
      const int64_t row = (int64_t)bh * Nq + g0 + sg * rows_per_sub + r;
      const int n = active ? max(0, min(row_count[row], cols_stride)) : 0;
      const int32_t* A = row_cols + row * cols_stride;
      for (int i = lane; i < n; i += 64) {
        const unsigned v = (unsigned)A[i];
        if (v < limit) atomicOr(&sub[wv][v >> 5], 1u << (v & 31));
      }
    }
    __syncthreads();
    for (int w = lane; w < words; w += 64) {
      const uint32_t x = sub[wv][w];
      uni_sub += __popc(x);
      bits[wv][w] |= x;                                  // word w belongs to this lane in every round
    }
  }
  int uni = 0;
  for (int w = lane; w < words; w += 64) uni += __popc(bits[wv][w]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    uni += __shfl_xor(uni, off);
    uni_sub += __shfl_xor(uni_sub, off);
  }
  if (active && lane == 0) {
    atomicAdd(&probe[0], uni);
    atomicAdd(&probe[1], uni_sub);
  }
}
template <int kB, int D>
basa_status attn_many(const SeqJob* seq, int n, const int64_t* out_strides, hipStream_t st) {
  {
    Jobs<TileJob<D>> jobs;
    for (int i = 0; i < n; ++i) {
      const SeqJob& s = seq[i];
      const int tiles = s.Nk * (kB / kTileKeys);
      jobs.add(TileJob<D>{s.k, s.v, s.perm_k, reinterpret_cast<uint4*>(s.tiles),
                          reinterpret_cast<uint4*>(s.tiles + sz_kv(s.k.heads, s.Nk, kB, D)), tiles},
               (int64_t)tiles * s.k.heads * 2);
    }
    ProfScope prof(K_GATHER, st);
    hipLaunchKernelGGL(many_kernel<TileJob<D>>, dim3(jobs.first[n]), dim3(256), 0, st, jobs);
    BASA_HIP_CHECK_LAUNCH("tile_kv");
  }
  // Workgroups of 128 or of 512 queries (same bits): the time of all of them by the step times of plan_call, over the
  // compute units, and the last ones to start, which find them unevenly full (the shortest: longest come first).  128 / 512,
  // whole batch, keep 50 %: 6 sequences of 565 to 7627 tokens, 16 heads: 783 / 756 us; 9 of 45000 in all: 1612 / 1549; kept
  // at 128: 10 of 6000, 8 heads: 82 / 107; 8 of 40000, 32 heads on 8, keep 25 %: 1628 / 1638; d = 64, where the narrow shape
  // hides its softmax better, 6 of 40000: 1000 / 1012.
  double solo_us = 0.0, wide_us = 0.0, tail_us = 0.0;
  for (int i = 0; i < n; ++i) {
    const SeqJob& s = seq[i];
    const double dead = 1.0 - (double)s.kappa / s.Nk, tiles = s.kappa * (kB / kTileKeys) * union_of_pair(kB, dead);
    const double scale = step_scale(D), wide_tiles = std::min((double)s.Nk * (kB / kTileKeys), tiles * union_of_groups(4, dead));
    solo_us += s.q.heads * ceil_div(s.Nq * kB, kSoloQueries) * (tiles * kSoloPairStepUs * scale + kSoloRoundUs) / 2.0;
    tail_us = wide_tiles * kWideStepUs * scale + kWideRoundUs;               // (ends at the shortest sequence)
    wide_us += s.q.heads * ceil_div(s.Nq * kB, kWideQueries) * tail_us;
  }
  const bool wide = D == 128 && wide_us / kCUs + tail_us < solo_us / kCUs;
  auto launch = [&](auto job, int queries, int qpw, bool fast, int stages) -> basa_status {
    typedef decltype(job) Job;
    constexpr bool kSolo = std::is_same<Job, AttnJob<kB, D>>::value;
    constexpr int kThreads = kSolo ? 256 : 512;
    constexpr auto kernel = &many_kernel<Job, kSolo ? 2 : 1, kThreads>;
    Jobs<Job> jobs;
    size_t lds = 0;
    for (int i = 0; i < n; ++i) {
      const SeqJob& s = seq[i];
      MfmaArgs m = {};
      m.q = s.q; m.Kt = s.tiles; m.Vt = s.tiles + sz_kv(s.k.heads, s.Nk, kB, D);
      m.row_count = s.row_count; m.row_cols = s.row_cols; m.cols_stride = s.kappa;
      m.perm_q = s.perm_q;
      m.out = reinterpret_cast<__bf16*>(s.out);
      m.out_sb = out_strides[0]; m.out_sh = out_strides[1]; m.out_sl = out_strides[2]; m.heads_q = s.q.heads;
      m.Nq = s.Nq; m.Nk = s.Nk; m.Lq = s.q.L; m.Lk = s.k.L;
      m.group = s.q.heads / s.k.heads;
      m.wgs_per_head = ceil_div(s.Nq * kB, queries);
      m.total_wgs = s.q.heads * m.wgs_per_head;
      m.scale_log2e = 1.4426950408889634f / sqrtf((float)D);
      m.splits = 1;
      m.stages = stages;
      m.redo = kSolo ? nullptr : s.redo;
      jobs.add(Job{m}, m.total_wgs);
      lds = std::max(lds, lds_bytes<D>(kThreads, qpw, s.Nk, false, fast, stages));
    }
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");
    ProfScope prof(K_ATTN, st);
    hipLaunchKernelGGL(kernel, dim3(jobs.first[n]), dim3(kThreads), lds, st, jobs);
    BASA_HIP_CHECK_LAUNCH("attn_mfma");
    return BASA_OK;
  };
  if (!wide) return launch(AttnJob<kB, D>{}, kSoloQueries, 32, true, 0);
  if constexpr (D == 128) {
    int longest = 0;
    for (int i = 0; i < n; ++i) longest = std::max(longest, seq[i].Nk);
    const basa_status e = launch(WideJob<kB, D, true>{}, kWideQueries, 64, true, wide_stages<D>(longest));
    return e != BASA_OK ? e : launch(WideJob<kB, D, false>{}, kWideQueries, 64, false, 2);
  }
  return BASA_OK;
}
}  // namespace

size_t attn_many_redo_bytes(int heads_q, int Lq, int B) { return (size_t)heads_q * ceil_div(ceil_div(Lq, B) * B, kWideQueries) * 4; }
size_t attn_many_tile_bytes(int heads_kv, int Lk, int d, int B) { return 2 * sz_kv(heads_kv, ceil_div(Lk, B), B, d); }
bool attn_many_takes(int Nk, int d) {
  // (the membership words of the key blocks live in the ring while the list is built; two workgroups per compute unit)
  return d == 128 ? (size_t)Nk * 4 <= 2 * Geo<128>::kStageBytes && lds_bytes<128>(256, 32, Nk, false, true) <= kLdsBytes / 2
                  : (size_t)Nk * 4 <= 2 * Geo<64>::kStageBytes && lds_bytes<64>(256, 32, Nk, false, true) <= kLdsBytes / 2;
}
basa_status launch_attn_many(const SeqJob* seq, int n, int B, const int64_t* out_strides, hipStream_t st) {
  if (seq[0].q.d == 128) return B == 128 ? attn_many<128, 128>(seq, n, out_strides, st) : attn_many<64, 128>(seq, n, out_strides, st);
  return B == 128 ? attn_many<128, 64>(seq, n, out_strides, st) : attn_many<64, 64>(seq, n, out_strides, st);
}

size_t attn_mfma_workspace_bytes(int BHq, int BHkv, int Lq, int Lk, int d, int B) {
  const int Nq = ceil_div(Lq, B), Nk = ceil_div(Lk, B);
  // + the two counters of the list-overlap probe + the key-index tiles of the causal variant
  // + one word per 512-query workgroup (which of them the pass with running maxima has to repeat)
  // + the bitmaps of the listed blocks
  return 2 * sz_kv(BHkv, Nk, B, d) + 256 + sz_kix(BHkv, Nk, B) + align_up((size_t)BHq * ceil_div(Nq * B, kWideQueries) * 4, 256) +
         sz_listed(BHkv, Nk);
}
size_t attn_mfma_split_bytes(int BHq, int Lq, int Lk, int d, int B, bool causal) {
  return align_up(part_bytes_of(BHq, Lq, ceil_div(Lk, B), B, d, causal), 256);
}

basa_status launch_attn_mfma(const AttnArgs& a, hipStream_t st) {
  const int BHq = a.q.batch * a.q.heads, BHkv = a.k.batch * a.k.heads;
  const int B = a.B;
  const int Nq = ceil_div(a.q.L, B), Nk = ceil_div(a.k.L, B);
  if (BHq == 0 || Nq == 0) return BASA_OK;
  const int d = a.q.d;
  {
    const size_t cap = d == 128 ? kMostBlocks<128> : kMostBlocks<64>;
    if ((size_t)Nk > cap) {
      set_error("attention: %d key blocks per head exceed the %zu this kernel can list (head dimension %d)", Nk, cap, d);
      return BASA_ERR_UNSUPPORTED;
    }
  }
  const size_t lds = d == 128 ? most_lds<128>(Nk) : most_lds<64>(Nk);
  {
    int dev = 0, max_lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute(shared memory per block)");
    if (lds > (size_t)max_lds) {
      set_error("attention needs %zu bytes of LDS for %d key blocks, the device offers %d", lds, Nk, max_lds);
      return BASA_ERR_UNSUPPORTED;
    }
  }
  char* ws = reinterpret_cast<char*>(a.ws);
  uint4* Kt = reinterpret_cast<uint4*>(ws);
  uint4* Vt = reinterpret_cast<uint4*>(ws + sz_kv(BHkv, Nk, B, d));
  int32_t* probe = reinterpret_cast<int32_t*>(ws + 2 * sz_kv(BHkv, Nk, B, d));
  int32_t* redo = reinterpret_cast<int32_t*>(ws + 2 * sz_kv(BHkv, Nk, B, d) + 256 + sz_kix(BHkv, Nk, B));

  int32_t* kix = a.causal ? reinterpret_cast<int32_t*>(ws + 2 * sz_kv(BHkv, Nk, B, d) + 256) : nullptr;
  MfmaArgs m;
  m.q = a.q; m.Kt = reinterpret_cast<const char*>(Kt); m.Vt = reinterpret_cast<const char*>(Vt);
  m.row_count = a.row_count; m.row_cols = a.row_cols; m.cols_stride = a.cols_stride;
  m.perm_q = a.perm_q;
  m.out = reinterpret_cast<__bf16*>(a.out); m.lse = a.lse;
  m.out_sb = a.out_sb; m.out_sh = a.out_sh; m.out_sl = a.out_sl; m.heads_q = a.q.heads;
  m.Nq = Nq; m.Nk = Nk; m.Lq = a.q.L; m.Lk = a.k.L;
  m.group = a.q.heads / a.k.heads;
  m.wgs_per_head = 0; m.total_wgs = 0;
  m.scale_log2e = 1.4426950408889634f / sqrtf((float)d);
  m.probe = nullptr; m.run_if_solo = 0; m.redo = nullptr;
  m.kix = kix; m.causal_off = a.causal_off;
  const int gsz = kWideQueries / B;
  Plan plan{false, 1, 0.0};
  m.stages = 0; m.splits = 1; m.part_o = nullptr; m.part_ml = nullptr;
  const int64_t rows = (int64_t)BHq * Nq * B;
  const bool small = rows < (int64_t)kSmallRounds * kCUs * kWideQueries;
  if (a.variant == 0 && rows < (int64_t)kPlannedRounds * kCUs * kWideQueries) {
    const size_t base = attn_mfma_workspace_bytes(BHq, BHkv, a.q.L, a.k.L, d, B);
    plan = plan_call(BHq, Nq, Nk, a.q.L, B, d, a.row_cols ? std::min(a.cols_stride, Nk) : Nk, a.causal != 0, small,
                     a.ws_bytes - base);
    if (plan.splits > 1) {
      m.splits = plan.splits;
      m.part_o = reinterpret_cast<float*>(ws + base);
      m.part_ml = reinterpret_cast<float2*>(m.part_o + (size_t)plan.splits * BHq * a.q.L * d);
    }
  }
  const bool can_probe = a.row_cols != nullptr && Nq >= 2 * gsz && (int64_t)BHq * Nq * B >= 2048 * 128;
  const bool solo_only = plan.solo && (small || !can_probe);
  const bool d64_alone = d == 64 && plan.splits == 1 && (int64_t)BHq * ceil_div(Nq * B, kSoloQueries) <= kCUs;
  const bool from_rows = solo_only && rows_pay(sz_kv(BHkv, Nk, B, d), plan.us, d64_alone) && offsets_fit(a.k.L, a.k.stride_l) &&
                         offsets_fit(a.v.L, a.v.stride_l);
  if (!from_rows) {
    ProfScope prof(K_GATHER, st);
    const dim3 grid(Nk * B / kTileKeys, BHkv, 2);
    const int by_index = a.causal && B == 128 && a.perm_k;
    const int rows = a.q.heads / a.k.heads * Nq;
    const int64_t entries = (int64_t)rows * a.cols_stride;
    uint32_t* listed = nullptr;
    int parts = 1;
    if (a.row_cols && entries < ((int64_t)1 << 31) && Nk <= 32 * kMaxListedWords &&
        bitmaps_pay(sz_kv(BHkv, Nk, B, d), std::min(1.0, (double)a.cols_stride / Nk), (double)entries * BHkv)) {
      parts = (int)std::min<int64_t>(std::min(rows, kListedParts), (entries + 4095) / 4096);
      listed = reinterpret_cast<uint32_t*>(ws + attn_mfma_workspace_bytes(BHq, BHkv, a.q.L, a.k.L, d, B) - sz_listed(BHkv, Nk));
      hipLaunchKernelGGL(listed_blocks_kernel, dim3(BHkv, parts), dim3(1024), 0, st, a.row_count, a.row_cols, a.cols_stride, rows,
                         Nk, listed);
      BASA_HIP_CHECK_LAUNCH("listed_blocks_kernel");
    }
    if (d == 128) hipLaunchKernelGGL(tile_kv_kernel<128>, grid, dim3(256), 0, st, a.k, a.v, a.perm_k, Kt, Vt, kix, probe, by_index,
                                    listed, parts, B / kTileKeys);
    else hipLaunchKernelGGL(tile_kv_kernel<64>, grid, dim3(256), 0, st, a.k, a.v, a.perm_k, Kt, Vt, kix, probe, by_index,
                                    listed, parts, B / kTileKeys);
    BASA_HIP_CHECK_LAUNCH("tile_kv_kernel");
  }
  if (a.causal) {
    if (plan.splits > 1) {
      ProfScope prof(K_ATTN, st);
      const basa_status s = launch_shape<kWideQueries, 64, true, false, true>(m, B, d, BHq, st);
      if (s != BASA_OK) return s;
    } else {
      ProfScope prof(K_ATTN, st);
      return launch_wide<true>(m, B, d, BHq, redo, a.variant != 4, st);
    }
    return launch_attn_combine(a, m.part_o, m.part_ml, m.splits, st);
  }
  if (solo_only) {
    {
      ProfScope prof(K_ATTN, st);
      const RowSource src{a.k, a.v, a.perm_k};
      const basa_status s = from_rows ? (plan.splits == 1 ? launch_rows<true, false>(m, src, B, d, BHq, st)
                                                          : launch_rows<false, true>(m, src, B, d, BHq, st))
                            : plan.splits == 1 ? launch_shape<kSoloQueries, 32, false, true>(m, B, d, BHq, st)
                                             : launch_shape<kSoloQueries, 32, false, false, true>(m, B, d, BHq, st);
      if (s != BASA_OK || plan.splits == 1) return s;
    }
    return launch_attn_combine(a, m.part_o, m.part_ml, m.splits, st);
  }

  // Which shape of workgroup: asked for, or (block lists given, enough work to pay for three tiny launches) decided on
  // the device from how much neighbouring lists overlap (plan.solo: between the two arithmetics of the 128-query shape,
  // so that the bits do not depend on which shape the plan takes for lists that overlap).
  int variant = a.variant;
  if (variant == 0 && !can_probe) variant = a.row_cols ? BASA_ATTN_DEFAULT_LISTS : 3;   // no lists: every block shares every tile
  if (variant == 0) {
    const int groups_total = BHq * (Nq / gsz);
    hipLaunchKernelGGL(list_overlap_kernel, dim3(ceil_div(ceil_div(groups_total, kProbeStride), 4)), dim3(256), 0, st,
                       a.row_count, a.row_cols, a.cols_stride, Nq, Nk, gsz, groups_total, probe);
    BASA_HIP_CHECK_LAUNCH("list_overlap_kernel");
    m.probe = probe;
  }
  ProfScope prof(K_ATTN, st);
  basa_status s = BASA_OK;
  if (variant == 1) return launch_shape<kSharedQueries, 32>(m, B, d, BHq, st);
  if (variant == 0 || variant == 3 || variant == 4) {
    m.run_if_solo = 0;
    s = plan.solo ? launch_shape<kSoloQueries, 32, false, true>(m, B, d, BHq, st)
                  : launch_wide<false>(m, B, d, BHq, redo, variant != 4, st);
    if (s != BASA_OK) return s;
  }
  if (variant == 0 || variant == 2) {
    m.run_if_solo = 1;
    s = launch_shape<kSoloQueries, 32>(m, B, d, BHq, st);
  }
  return s;
}

}  // namespace basa
