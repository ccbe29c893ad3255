// Block-sparse attention for f32 tensors (Sec. 2; Eq. 1; Alg. 1 step 12): inputs, accumulation and softmax
// state in fp32 throughout.  Two kernels: on the fp32 matrix instruction (small calls, the causal variant, workspaces
// without room, and whatever holds infinities or huge numbers), and on the bf16 one with every number as the exact sum of three (below).
//
// The fp32 instruction.
// Bound: the matrix cores.  v_mfma_f32_32x32x2_f32 does 4096 flop in 64 cycles (157 TFLOP/s over
// the chip); a 32-key tile costs a wave of 32 queries 2 x D/2 of them, 8192 cycles at D = 128, against
// about 500 cycles of softmax arithmetic and 32 16-byte LDS reads.
//
// A workgroup owns 32 QG queries of ONE query block and walks that block's own list (no union, no
// idle waves).  Its waves are QG query groups x KS key slices: slice s takes every KS-th 32-key tile,
// with an online softmax of its own, and the slices are merged through LDS at the end.  Slices
// rather than more queries per workgroup: two waves per SIMD hide each other's softmax, and a map
// with few query blocks still occupies the chip.  When it does not (few heads, short sequences, or a
// last round of workgroups that is mostly empty) the list is further split over `splits` workgroups,
// whose partial results attn_combine_kernel adds up.
//
// K and V rows are gathered straight from the caller's tensors, through perm_k, by direct-to-LDS
// loads (the source address of a lane is free, its LDS slot is not): no tiling pass, one launch.  The
// scores are computed transposed, S^T = K Q^T, so that a lane owns one query (running maximum and
// sum are per-lane scalars) and register r of the score accumulator is, as it stands, the B operand of
// the second product's step r (O^T += V^T P^T, two keys per step): no conversion, no lane exchange.
// Row i of output block db is dimension (D/32) i + db, so that one 16-byte read of a V row feeds
// the matrix instruction of all four output blocks (8 bytes, two blocks, at D = 64).  K: 16-byte chunk
// c of row r sits at c ^ (r & 15), V is linear: both conflict-free.
//
// Measured (8 heads, L = 4096, d = B = 128, 16 of 32 blocks): 3037 us for the former kernel (one
// thread per query, fp32 FMA) -> 293 us, 117 TFLOP/s of the 154 the library's fp32 matrix product
// reaches on this card (the matrix cores are busy 75 % of the cycles; the vector instructions of a tile are
// only partly hidden behind them, and two independent workgroups per compute unit instead of two slices
// that meet at a barrier measure the same); one head, L = 1024, d = B = 64: 345 -> 12 + 4 us.
#include <algorithm>
#include <climits>
#include <cstdint>
#include "common.hpp"

namespace basa {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

constexpr int kTK = 32;                     // keys per tile
constexpr float kLazyTau = 8.0f;            // log2 of the largest exponentiated score kept before a rescale
constexpr int kCUs = 256, kMaxSplits = 16;
constexpr size_t kLdsBytes = 160 * 1024;

// Log-sum-exp from a running maximum in log2 units and its sum.  The unit is the rounded scale_log2e times a score, so
// the factor back to natural units is computed from it in double and kept in two parts, and the sum m + log2(l), whose
// last place is twice that of the result, is not formed: scores near 1000 (lse 2000, d = 64): off by 8.7e-5 at
// most, 1.8e-4 as (m + log2(l)) ln 2; half a unit in the last place is 6.1e-5.
struct LseFactor { float hi, lo; };
LseFactor lse_factor(int d) {
  const double f = 1.0 / (sqrt((double)d) * (double)(1.4426950408889634f / sqrtf((float)d)));
  LseFactor k;
  k.hi = (float)f; k.lo = (float)(f - (double)k.hi);
  return k;
}
__device__ __forceinline__ float lse_of(float m, float l, LseFactor k) {
  return l == 0.f ? -INFINITY : fmaf(m, k.hi, fmaf(m, k.lo, __log2f(l) * 0.6931471805599453f));
}

struct F32Args {
  AttnArgs a;
  int Nq, Nk, group, wgs_per_head, total, splits;
  float scale_log2e;
  LseFactor lse_k;
  float* part_o;                            // splits > 1: [split][BHq][Lq][D], rows by sorted position
  float2* part_ml;                          //             [split][BHq][Lq] running maximum (log2), running sum
  const int32_t* redo;                      // kRedo: [BHq][redo_wgs]: the 128 queries whose rows are wanted (1)
  int redo_wgs;
};

// kRedo: only the workgroups that p.redo marks.
template <int D, int QG, int KS, bool kCausal, bool kRedo>
__global__ __launch_bounds__(64 * QG * KS, QG * KS == 8 ? 2 : 1) void attn_f32_kernel(F32Args p) {
  constexpr int CPR = D / 4;                // 16-byte chunks per row
  constexpr int DB = D / 32;                // output blocks of 32 dimensions
  constexpr int kHalf = kTK * D * 4;        // bytes of a K tile (and of a V tile)
  constexpr int kStage = 2 * kHalf;
  constexpr int kChunks = kHalf / 1024;     // wave-wide loads per K tile
  static_assert(kChunks % QG == 0, "the chunks of a tile are dealt to the waves of its slice in rounds");
  extern __shared__ __attribute__((aligned(16))) char smem[];   // [slice][stage][K tile, V tile], then key indices
  int* kix = reinterpret_cast<int*>(smem + KS * 2 * kStage);    // kCausal: [slice][stage][kTK] original key indices

  const AttnArgs& a = p.a;
  int logical = blockIdx.x;                 // one XCD, one range of heads
  if ((p.total & 7) == 0) logical = (blockIdx.x & 7) * (p.total >> 3) + (blockIdx.x >> 3);
  const int split = logical % p.splits;
  const int wgi = logical / p.splits;
  const int bhq = wgi / p.wgs_per_head, wg = wgi - bhq * p.wgs_per_head;
  if constexpr (kRedo) {
    if (p.redo[bhq * p.redo_wgs + wg * (32 * QG) / 128] == 0) return;
  }
  const int bhk = bhq / p.group;
  const int lane = threadIdx.x & 63, li = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = wave % QG, slice = wave / QG;
  const int Lq = a.q.L, Lk = a.k.L, B = a.B;
  const int pos = wg * (32 * QG) + g * 32 + li;          // sorted position of this lane's query
  const int gq = wg * (32 * QG) / B;
  const int qrow = pos < Lq ? perm_at(a.perm_q, (int64_t)bhq * Lq, pos, Lq) : 0;
  const int q_lim = (kCausal && pos < Lq) ? qrow + a.causal_off : INT_MIN;

  const int64_t rowid = (int64_t)bhq * p.Nq + gq;
  const int count = a.row_cols ? min(a.row_count[rowid], a.cols_stride) : p.Nk;
  const int32_t* cols = a.row_cols ? a.row_cols + rowid * a.cols_stride : nullptr;
  const int tpb = B / kTK, tiles = max(0, count) * tpb;
  const int stride = p.splits * KS, first = split * KS + slice;
  const int steps = (tiles + stride - 1) / stride;
  const int32_t* pk = a.perm_k ? a.perm_k + (int64_t)bhk * Lk : nullptr;
  const char* kbase = reinterpret_cast<const char*>(a.k.ptr) + a.k.head_offset(bhk) * 4;
  const char* vbase = reinterpret_cast<const char*>(a.v.ptr) + a.v.head_offset(bhk) * 4;
  char* ring = smem + slice * 2 * kStage;

  // First key of this slice's tile of step s, or -1: past the list, not a key block, or past the last
  // key.  Lane l holds the one of step 64 n + l, read for 64 steps at a time: a list entry loaded step by step
  // would be waited for behind the tile loads that are in flight.
  auto keys_of_64_steps = [&](int s0) -> int {
    const int i = (s0 + lane) * stride + first;
    // (loaded before the count is known: the list, the count and perm_q then arrive together)
    const int gk = cols ? cols[min(i / tpb, a.cols_stride - 1)] : i / tpb;
    const int key0 = gk * B + (i % tpb) * kTK;
    return (i < tiles && (unsigned)gk < (unsigned)p.Nk && key0 < Lk) ? key0 : -1;
  };
  // Original index of key li of the tile (clamped: a key past the end is masked where it is used), as stored:
  // perm_at's check is made when it is used, one step later, so that nothing waits for the load here.
  auto raw_row = [&](int key0) -> int {
    const int kp = min(max(key0, 0) + li, Lk - 1);
    return pk ? pk[kp] : kp;
  };
  // row * stride * 4 with one 32 x 32 -> 64 bit multiply (the high half of a stride is nearly always 0)
  auto row_bytes = [&](uint32_t row, int64_t stride) -> uint64_t {
    const uint64_t sb = (uint64_t)stride * 4;
    uint64_t off = (uint64_t)row * (uint32_t)sb;
    if (sb >> 32) off += (uint64_t)(row * (uint32_t)(sb >> 32)) << 32;
    return off;
  };
  auto issue = [&](int key0, int raw, int stage) {
    if (key0 < 0) return;
    const int rows = (unsigned)raw < (unsigned)Lk ? raw : min(key0 + li, Lk - 1);
    char* dst = ring + stage * kStage;
#pragma unroll
    for (int j = 0; j < kChunks / QG; ++j) {
      const int ch = j * QG + g;
      const int r = ch * (64 / CPR) + lane / CPR, c = lane % CPR;
      const uint32_t row = (uint32_t)__shfl(rows, r);
      const char* ks = kbase + row_bytes(row, a.k.stride_l) + 16 * (c ^ (r & 15));
      const char* vs = vbase + row_bytes(row, a.v.stride_l) + 16 * c;
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)ks, (lds_ptr_t)(dst + ch * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)vs, (lds_ptr_t)(dst + kHalf + ch * 1024), 16, 0, 0);
    }
    if (kCausal && g == 0 && lane < kTK) kix[(slice * 2 + stage) * kTK + lane] = key0 + lane < Lk ? rows : INT_MAX;
  };

  int keys = keys_of_64_steps(0);
  int key_cur = __builtin_amdgcn_readlane(keys, 0), key_nxt = __builtin_amdgcn_readlane(keys, 1);
  {
    const int raw0 = raw_row(key_cur);
    issue(key_cur, raw0, 0);
  }
  int raw_nxt = raw_row(key_nxt);
  floatx4 qf[D / 8];                        // lane (query li, half h): Q[8 k + 4 h .. + 3]
  {
    const floatx4* qp = reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(a.q.ptr) + a.q.head_offset(bhq) +
                                                         (int64_t)qrow * a.q.stride_l);
#pragma unroll
    for (int k = 0; k < D / 8; ++k) qf[k] = qp[2 * k + h];
  }
  floatx16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = floatx16{0};
  float m_run = -INFINITY, l_run = 0.f;
  const float c = p.scale_log2e;
  // The two waves of a SIMD belong to different halves of the slices: one half asks for its next tile before
  // the first product, the other after it, so that the two do not run through softmax and address
  // arithmetic in step while the matrix core idles.
  const bool late = slice >= KS / 2;

  for (int s = 0; s < steps; ++s) {
    // my loads of step s have landed (and the key rows of step s + 1); after the barrier everyone's have,
    // and everyone is done with the other stage, which the next loads overwrite
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    const int stage = s & 1;
    int key_n2 = -1, raw_n2 = 0;
    auto next_tile = [&]() {
      issue(key_nxt, raw_nxt, stage ^ 1);
      if (((s + 2) & 63) == 0) keys = keys_of_64_steps(s + 2);
      key_n2 = __builtin_amdgcn_readlane(keys, (s + 2) & 63);
      raw_n2 = raw_row(key_n2);
    };
    if (!late || key_cur < 0) next_tile();
    if (key_cur >= 0) {
      const char* ks = ring + stage * kStage;
      const char* vs = ks + kHalf;
      floatx16 sc = floatx16{0};
#pragma unroll
      for (int k = 0; k < D / 8; ++k) {
        const floatx4 kf = *reinterpret_cast<const floatx4*>(ks + li * (D * 4) + (((2 * k + h) ^ (li & 15)) << 4));
#pragma unroll
        for (int j = 0; j < 4; ++j) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j], qf[k][j], sc, 0, 0, 0);
      }
      if (late) next_tile();
      if (key_cur + kTK > Lk) {
        // Rows past the end hold copies of the last one; their probabilities are 0, but 0 times an infinity of V
        // is not.  Every wave clears all of them itself (its own reads come after its own writes).
        const char* v0 = vs + (Lk - key_cur) * (D * 4);
        for (int i = lane; i < (key_cur + kTK - Lk) * CPR; i += 64)
          reinterpret_cast<floatx4*>(const_cast<char*>(v0))[i] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      // register r of half h: key 8 (r / 4) + 4 h + r % 4 of the tile
      if constexpr (kCausal) {
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int4 ix = *reinterpret_cast<const int4*>(kix + (slice * 2 + stage) * kTK + 8 * r4 + 4 * h);
          if (ix.x > q_lim) sc[4 * r4] = -INFINITY;
          if (ix.y > q_lim) sc[4 * r4 + 1] = -INFINITY;
          if (ix.z > q_lim) sc[4 * r4 + 2] = -INFINITY;
          if (ix.w > q_lim) sc[4 * r4 + 3] = -INFINITY;
        }
      } else if (key_cur + kTK > Lk) {
        const int nvalid = Lk - key_cur;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + 4 * h + (r & 3) >= nvalid) sc[r] = -INFINITY;
      }
      float mx = sc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
      if (__builtin_amdgcn_ballot_w64(mx > m_run + kLazyTau) != 0) {
        const float m_new = fmaxf(m_run, mx);
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      }
      // (a query that has seen no finite score yet subtracts 0, so that exp2 sees -inf, never inf - inf)
      const float m_use = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], c, -m_use));
        l_run += sc[r];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const char* vrow = vs + (8 * (r >> 2) + 4 * h + (r & 3)) * (D * 4) + li * (4 * DB);
        if constexpr (DB == 4) {
          const floatx4 vf = *reinterpret_cast<const floatx4*>(vrow);
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db], sc[r], o[db], 0, 0, 0);
        } else {
          const floatx2 vf = *reinterpret_cast<const floatx2*>(vrow);
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db], sc[r], o[db], 0, 0, 0);
        }
      }
    }
    key_cur = key_nxt; key_nxt = key_n2; raw_nxt = raw_n2;
  }

  // ---- merge the key slices through LDS (the ring is free once everyone has left the loop)
  float l_tot = l_run + __shfl_xor(l_run, 32);
  asm volatile("" : "+v"(l_tot));           // (the lane exchange is over before the barriers below)
  if constexpr (KS > 1) {
    constexpr int kSlot = DB * 16 * 64 * 4 + 2 * 64 * 4;           // one wave's accumulators, then its maxima and sums
    static_assert((KS - 1) * QG * kSlot <= KS * 2 * kStage, "the slices' results fit the ring");
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (slice > 0) {
      float* w = reinterpret_cast<float*>(smem + ((slice - 1) * QG + g) * kSlot);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          reinterpret_cast<floatx4*>(w)[(db * 4 + r4) * 64 + lane] =
              floatx4{o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]};
      w[DB * 16 * 64 + lane] = m_run;
      w[DB * 16 * 64 + 64 + lane] = l_tot;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (slice > 0) return;
#pragma unroll
    for (int s = 1; s < KS; ++s) {
      const float* w = reinterpret_cast<const float*>(smem + ((s - 1) * QG + g) * kSlot);
      const float ms = w[DB * 16 * 64 + lane], ls = w[DB * 16 * 64 + 64 + lane];
      const float m_new = fmaxf(m_run, ms);
      const float f0 = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      const float f1 = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - m_new);
      l_tot = l_tot * f0 + ls * f1;
      m_run = m_new;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const floatx4 t = reinterpret_cast<const floatx4*>(w)[(db * 4 + r4) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[db][4 * r4 + e] = o[db][4 * r4 + e] * f0 + t[e] * f1;
        }
    }
  }
  if (pos >= Lq) return;
  // register r of block db: dimension DB i + db, i = 8 (r / 4) + 4 h + r % 4
  if (p.splits > 1) {
    const int64_t prow = ((int64_t)split * (p.total / (p.splits * p.wgs_per_head)) + bhq) * Lq + pos;
    float* po = p.part_o + prow * D;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 8 * (r >> 2) + 4 * h + (r & 3);
      if constexpr (DB == 4) *reinterpret_cast<floatx4*>(po + 4 * i) = floatx4{o[0][r], o[1][r], o[2][r], o[3][r]};
      else *reinterpret_cast<floatx2*>(po + 2 * i) = floatx2{o[0][r], o[1][r]};
    }
    if (h == 0) p.part_ml[prow] = make_float2(m_run, l_tot);
    return;
  }
  const float inv_l = l_tot > 0.f ? 1.0f / l_tot : 0.f;            // a row without any visible key: zeros
  float* op = reinterpret_cast<float*>(a.out) + a.out_offset(bhq, qrow);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = 8 * (r >> 2) + 4 * h + (r & 3);
    if constexpr (DB == 4) *reinterpret_cast<floatx4*>(op + 4 * i) = floatx4{o[0][r], o[1][r], o[2][r], o[3][r]} * inv_l;
    else *reinterpret_cast<floatx2*>(op + 2 * i) = floatx2{o[0][r], o[1][r]} * inv_l;
  }
  if (a.lse && h == 0) a.lse[(int64_t)bhq * Lq + qrow] = lse_of(m_run, l_tot, p.lse_k);
}

// ---------------------------------------------------------------------------------------------
// The same on the bf16 matrix instruction, for calls with enough work: every fp32 number is the exact sum of
// three bf16 numbers (24 bits as 8 + 8 + 8, each part rounded to nearest), products of two of those are exact in fp32, and the six part
// products above 2^-24 of a product are accumulated in fp32, the small ones first: 6 x 32 cycles per 32 x 32 x 16
// against 8 x 64 of v_mfma_f32_32x32x2_f32.  The probabilities are cut up in registers, K and V once per call by
// split_kv_kernel, which leaves the LDS image of every tile (two tiles of 32 keys, K and V^T, three parts: 96 KB at
// D = 128).
//
// A workgroup owns 128 queries (one query block of 128, two of 64, whose lists it walks together), one wave per 32 of
// them and key slice; the two slices of a SIMD are half a tile apart: one multiplies K Q^T while the other
// exponentiates and multiplies V^T P^T, so that the matrix cores have work while the vector unit does, and every LDS
// buffer is refilled in the half in which nobody reads it.
//
// Parts of small numbers would be subnormal bf16 and lose bits (from 2^-110 down), so what the rows are made of is cut up in
// larger units, V times 2^24 and the probabilities times 2^24: the parts of every fp32 number are exact then, and the rows are
// scaled back at the end.  (Powers of two: ordinary inputs keep their bits.  V of 1e-36: 2.7e-5 off 64 bits without, 3.4e-7
// with; rows that only probabilities of 2^-124 make up: 3.4e-4 -> 1.9e-6, as the fp32 instruction; time +0.3 %.)  In a number
// of K or Q an error of 2^-126 matters only where the other factor is huge, and parts of numbers of 2^86 and more are NaN.
//
// A part of a huge number, an infinity or a NaN, or of a product or sum that overflows, is NaN or turns into it, and it reaches
// the sum or the row of every query it touches: such a workgroup writes one word, and attn_f32_kernel, launched behind this
// one, computes its rows instead (and returns at once elsewhere).
//
// Bound: power and the vector unit (306 instructions a tile next to 96 MFMAs; 1.16 PFLOP/s of part products with every
// compute unit busy; without the tile loads 6 % faster).  8 heads, L = 4096, d = B = 128, 16 of 32 blocks: 276 us on
// the fp32 instruction -> 177 us + 13.5 us for the tiles; error against 64 bits 6.4e-7 -> 2.7e-7 (2-norm), largest 1.5e-5 ->
// 0.8e-5 of the root mean square: the probabilities and the scores are rounded as before, their sums less often.
// ---------------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));

template <int D>
struct SplitGeo {
  static constexpr int kRow = D * 2;                 // bytes of a K row of one part
  static constexpr int kPart = kTK * D * 2;          // one part of a K or V^T tile
  static constexpr int kBuf = 3 * kPart;             // K tile; a V^T tile is as large
  static constexpr int kTile = 2 * kBuf;
  // 16 consecutive rows of K, or of V^T (64 bytes each), read at one chunk hit 16 distinct 16-byte bank groups
  static __device__ __forceinline__ int k_chunk(int row, int c) { return c ^ (D == 128 ? row & 15 : (row >> 1) & 7); }
  static __device__ __forceinline__ int v_chunk(int row, int c) { return c ^ ((row >> 2) & 3); }
};

constexpr float kUnit = 16777216.f, kPerUnit = 1.f / kUnit;       // 2^24
constexpr float kHuge = 7.7371252e25f;                            // 2^86

// Two floats into their three parts, packed in pairs (low half: a).
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& w0, uint32_t& w1, uint32_t& w2) {
  auto pack = [](float x, float y) { return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)x, (__bf16)y}); };
  w0 = pack(a, b);
  const float ra = a - __uint_as_float(w0 << 16), rb = b - __uint_as_float(w0 & 0xffff0000u);
  w1 = pack(ra, rb);
  w2 = pack(ra - __uint_as_float(w1 << 16), rb - __uint_as_float(w1 & 0xffff0000u));
}
__device__ __forceinline__ void split8(const floatx4& x, const floatx4& y, uintx4 (&w)[3]) {
  uint32_t a, b, c;
  split_pair(x[0], x[1], a, b, c); w[0][0] = a; w[1][0] = b; w[2][0] = c;
  split_pair(x[2], x[3], a, b, c); w[0][1] = a; w[1][1] = b; w[2][1] = c;
  split_pair(y[0], y[1], a, b, c); w[0][2] = a; w[1][2] = b; w[2][2] = c;
  split_pair(y[2], y[3], a, b, c); w[0][3] = a; w[1][3] = b; w[2][3] = c;
}
// Numbers of Q or K whose products the parts of small factors would not be exact enough for become NaN.
__device__ __forceinline__ floatx4 not_huge(floatx4 x) {
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = fabsf(x[e]) < kHuge ? x[e] : __uint_as_float(0x7fc00000u);
  return x;
}

// One 32-key tile of a KV head, blockIdx.z = 0 its K rows, 1 its V rows transposed; rows past the end are zeros.  Bound
// by memory: 4 bytes read and 6 written per element.
template <int D>
__global__ __launch_bounds__(256) void split_kv_kernel(TensorView k, TensorView v, const int32_t* __restrict__ perm,
                                                       char* __restrict__ img, int32_t* __restrict__ redo, int redo_words) {
  using G = SplitGeo<D>;
  constexpr int CPR = D / 8, kItems = kTK * CPR / 256;         // 8 numbers (a chunk of every part) to a thread and item
  __shared__ __attribute__((aligned(16))) uint16_t cols[3][kTK][D + 8];
  const int tile = blockIdx.x, bh = blockIdx.y, t = threadIdx.x;
  const bool is_v = blockIdx.z != 0;
  if (tile == 0 && bh == 0 && !is_v)
    for (int i = t; i < redo_words; i += 256) redo[i] = 0;
  const TensorView& x = is_v ? v : k;
  const char* base = reinterpret_cast<const char*>(x.ptr) + x.head_offset(bh) * 4;
  const int32_t* pm = perm ? perm + (int64_t)bh * x.L : nullptr;
  char* dst = img + ((int64_t)bh * gridDim.x + tile) * G::kTile;
  int row[kItems];
  floatx4 lo[kItems], hi[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int pos = min(tile * kTK + (it * 256 + t) / CPR, x.L - 1);
    row[it] = pm ? pm[pos] : pos;
  }
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int pos = min(tile * kTK + (it * 256 + t) / CPR, x.L - 1), r = (unsigned)row[it] < (unsigned)x.L ? row[it] : pos;
    const floatx4* src = reinterpret_cast<const floatx4*>(base + (int64_t)r * x.stride_l * 4) + 2 * ((it * 256 + t) % CPR);
    lo[it] = src[0];
    hi[it] = src[1];
  }
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int id = it * 256 + t, r = id / CPR, c = id % CPR;
    if (tile * kTK + r >= x.L) lo[it] = hi[it] = floatx4{0.f, 0.f, 0.f, 0.f};
    uintx4 w[3];
    if (is_v) split8(lo[it] * kUnit, hi[it] * kUnit, w);
    else split8(not_huge(lo[it]), not_huge(hi[it]), w);
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      if (!is_v) *reinterpret_cast<uintx4*>(dst + part * G::kPart + r * G::kRow + 16 * G::k_chunk(r, c)) = w[part];
      else *reinterpret_cast<uintx4*>(&cols[part][r][8 * c]) = w[part];
    }
  }
  if (!is_v) return;                                 // uniform
  __syncthreads();
  // chunk s of row d: keys 16 (s / 2) + 8 (e / 4) + 4 (s % 2) + e % 4, the order in which the second product finds the
  // scores of a lane
#pragma unroll
  for (int it = 0; it < 3 * D * 4 / 256; ++it) {
    const int id = it * 256 + t, part = id / (D * 4), dd = id / 4 % D, s = id % 4;
    uint32_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = cols[part][16 * (s >> 1) + 8 * (j >> 2) + 4 * (s & 1) + (j & 3)][dd];
    *reinterpret_cast<uintx4*>(dst + G::kBuf + part * G::kPart + dd * 64 + 16 * G::v_chunk(dd, s)) =
        uintx4{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
  }
}

struct SplitArgs {
  AttnArgs a;
  int Nq, Nk, group, wgs_per_head, total, splits;
  float scale_log2e;
  LseFactor lse_k;
  const char* img;                          // [BHkv][tile of 32 keys][K parts, V^T parts]
  int32_t* redo;                            // [BHq][wgs_per_head]: 1 = left to attn_f32_kernel
  float* part_o;                            // as in F32Args
  float2* part_ml;
};

template <int D, int kB>
__global__ __launch_bounds__(512) void attn_split_kernel(SplitArgs p) {
  using G = SplitGeo<D>;
  constexpr int kSteps = D / 16, DB = D / 32, NQB = 128 / kB, TPB = kB / kTK, kChunks = G::kBuf / 1024;
  static_assert(kChunks % 4 == 0, "the chunks of a tile are dealt to the four waves of its slice");
  extern __shared__ __attribute__((aligned(16))) char smem[];   // [slice][K tile, V^T tile], list, counts
  uint32_t* flags = reinterpret_cast<uint32_t*>(smem);          // (while the list is built)
  uint32_t* seq = reinterpret_cast<uint32_t*>(smem + 2 * G::kTile);
  uint32_t* wave_counts = seq + p.Nk;
  const AttnArgs& a = p.a;
  int logical = blockIdx.x;                 // one XCD, one range of heads
  if ((p.total & 7) == 0) logical = (blockIdx.x & 7) * (p.total >> 3) + (blockIdx.x >> 3);
  const int split = logical % p.splits, wgi = logical / p.splits;
  const int bhq = wgi / p.wgs_per_head, wg = wgi - bhq * p.wgs_per_head;
  const int bhk = bhq / p.group;
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = wave & 3, slice = wave >> 2;
  const int Lq = a.q.L, Lk = a.k.L;
  const int pos = wg * 128 + g * 32 + li;                // sorted position of this lane's query
  const int qrow = pos < Lq ? perm_at(a.perm_q, (int64_t)bhq * Lq, pos, Lq) : 0;
  const floatx4* qp = reinterpret_cast<const floatx4*>(reinterpret_cast<const float*>(a.q.ptr) + a.q.head_offset(bhq) +
                                                       (int64_t)qrow * a.q.stride_l);

  // ---- the union of the query blocks' lists, ascending; bit 24 + b: query block b of the workgroup lists the block
  const int nqb = min(NQB, p.Nq - wg * NQB);
  for (int c = tid; c < p.Nk; c += 512) flags[c] = a.row_cols ? 0u : (1u << nqb) - 1u;
  __syncthreads();
  if (a.row_cols) {
    for (int b = 0; b < nqb; ++b) {
      const int64_t rowid = (int64_t)bhq * p.Nq + wg * NQB + b;
      const int cnt = min(a.row_count[rowid], a.cols_stride);
      for (int i = tid; i < cnt; i += 512) {
        const int col = a.row_cols[rowid * a.cols_stride + i];
        if ((unsigned)col < (unsigned)p.Nk) atomicOr(&flags[col], 1u << b);
      }
    }
    __syncthreads();
  }
  int n_union = 0;
  for (int base = 0; base < p.Nk; base += 512) {
    const int c = base + tid;
    const uint32_t f = c < p.Nk ? flags[c] : 0u;
    const uint64_t bal = __builtin_amdgcn_ballot_w64(f != 0u);
    if (lane == 0) wave_counts[wave] = __popcll(bal);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const int cw = wave_counts[w];
      before += w < wave ? cw : 0;
      total += cw;
    }
    if (f != 0u) seq[n_union + before + __popcll(bal & ((1ull << lane) - 1ull))] = (uint32_t)c | f << 24;
    n_union += total;
    __syncthreads();
  }
  int n_tiles = n_union * TPB;
  if (n_union > 0) {                         // tiles of the last key block that hold no key
    const int key0 = (int)(seq[n_union - 1] & 0xffffffu) * kB;
    n_tiles -= TPB - min(TPB, (Lk - key0 + kTK - 1) / kTK);
  }
  const int stride = p.splits * 2, first = split * 2 + slice, steps = (n_tiles + stride - 1) / stride;
  const char* head = p.img + (int64_t)bhk * (p.Nk * TPB) * G::kTile;
  char* kbuf = smem + slice * G::kTile;
  char* vbuf = kbuf + G::kBuf;
  auto entry_of = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)seq[min(i, n_tiles - 1) / TPB]); };
  // a K or V^T tile (at `part_of_tile` of tile i's image) into `dst` by the four waves of the slice
  auto issue = [&](uint32_t e, int i, int part_of_tile, char* dst) {
    const char* src = head + (int64_t)((int)(e & 0xffffffu) * TPB + i % TPB) * G::kTile + part_of_tile;
#pragma unroll
    for (int j = 0; j < kChunks / 4; ++j) {
      const int ch = j * 4 + g;
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(src + ch * 1024 + (uint32_t)(lane * 16)), (lds_ptr_t)(dst + ch * 1024), 16, 0, 0);
    }
  };

  floatx16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) o[db] = floatx16{0};
  float m_run = -INFINITY, l_run = 0.f;
  const float c = p.scale_log2e;
  const uint32_t my_bit = 1u << (24 + g * 32 / kB);
  if (n_tiles > 0) {
    uint32_t e_cur = entry_of(first);
    if (first < n_tiles) issue(e_cur, first, 0, kbuf);
    bf16x8 qf[3][kSteps];                     // lane (query li, half h): parts of Q[16 s + 8 h .. + 7]
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      uintx4 w[3];
      split8(not_huge(qp[4 * s + 2 * h]), not_huge(qp[4 * s + 2 * h + 1]), w);
#pragma unroll
      for (int part = 0; part < 3; ++part) qf[part][s] = __builtin_bit_cast(bf16x8, w[part]);
    }
    if (slice == 1) __syncthreads();
    for (int t = 0; t < steps; ++t) {
      const int i = t * stride + first;
      const bool mine = i < n_tiles && (e_cur & my_bit);
      const int key0 = ((int)(e_cur & 0xffffffu) * TPB + i % TPB) * kTK;
      // K of tile i has landed, and the slice is done with the V of the one before
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();
      if (i < n_tiles) issue(e_cur, i, G::kBuf, vbuf);
      const uint32_t e_nxt = entry_of(i + stride);
      floatx16 sc = floatx16{0};
      if (mine) {
        // Fragments of a step are read while the matrix cores are at the step before (the fences keep the compiler
        // from moving the reads down again).  The small products have an accumulator of their own.
        auto k_frags = [&](int s, bf16x8 (&f)[3]) {
#pragma unroll
          for (int part = 0; part < 3; ++part)
            f[part] = *reinterpret_cast<const bf16x8*>(kbuf + part * G::kPart + li * G::kRow + 16 * G::k_chunk(li, 2 * s + h));
        };
        bf16x8 kf[2][3];
        floatx16 lo = floatx16{0};
        k_frags(0, kf[0]);
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
          if (s + 1 < kSteps) k_frags(s + 1, kf[(s + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          const bf16x8(&f)[3] = kf[s & 1];
          lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[2], qf[0][s], lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], qf[1][s], lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], qf[2][s], lo, 0, 0, 0);
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], qf[0][s], sc, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], qf[0][s], lo, 0, 0, 0);
          lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], qf[1][s], lo, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] += lo[r];
        // register r of half h: key 8 (r / 4) + 4 h + r % 4 of the tile
        if (key0 + kTK > Lk) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (8 * (r >> 2) + 4 * h + (r & 3) >= Lk - key0) sc[r] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * c;
        if (__builtin_amdgcn_ballot_w64(mx > m_run + kLazyTau) != 0) {
          const float m_new = fmaxf(m_run, mx);
          const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
          m_run = m_new;
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
        }
        const float m_use = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], c, -m_use)) * kUnit;
          l_run += sc[r];
        }
      }
      // V^T of tile i has landed, and the slice is done with its K
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __syncthreads();
      if (i + stride < n_tiles) issue(e_nxt, i + stride, 0, kbuf);
      if (mine) {
        auto v_frags = [&](int n, bf16x8 (&f)[3]) {
#pragma unroll
          for (int part = 0; part < 3; ++part)
            f[part] = *reinterpret_cast<const bf16x8*>(vbuf + part * G::kPart + (32 * (n >> 1) + li) * 64 +
                                                       16 * G::v_chunk(li, 2 * (n & 1) + h));
        };
        // (a tile's own sum first, which keeps the rounding of the row at one per tile: 2.7e-7 instead of 4.6e-7 off 64
        //  bits in the workload above, for 1.5 % of the time)
        bf16x8 vf[2][3], pf[2][3];
        floatx16 t = floatx16{0};
        v_frags(0, vf[0]);
#pragma unroll
        for (int gr = 0; gr < 2; ++gr) {
          uintx4 w[3];
          split8(floatx4{sc[8 * gr], sc[8 * gr + 1], sc[8 * gr + 2], sc[8 * gr + 3]},
                 floatx4{sc[8 * gr + 4], sc[8 * gr + 5], sc[8 * gr + 6], sc[8 * gr + 7]}, w);
#pragma unroll
          for (int part = 0; part < 3; ++part) pf[gr][part] = __builtin_bit_cast(bf16x8, w[part]);
        }
#pragma unroll
        for (int n = 0; n < 2 * DB; ++n) {
          if (n + 1 < 2 * DB) v_frags(n + 1, vf[(n + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          const bf16x8(&f)[3] = vf[n & 1];
          const bf16x8(&x)[3] = pf[n & 1];
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[2], x[0], t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], x[1], t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], x[2], t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[1], x[0], t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], x[1], t, 0, 0, 0);
          t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[0], x[0], t, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (n & 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) o[n >> 1][r] += t[r];
            t = floatx16{0};
          }
        }
      }
      e_cur = e_nxt;
    }
    if (slice == 0) __syncthreads();
  }

  // ---- merge the two slices through LDS
  float l_tot = l_run + __shfl_xor(l_run, 32);
  asm volatile("" : "+v"(l_tot));
  constexpr int kSlot = DB * 16 * 64 * 4 + 2 * 64 * 4;
  static_assert(4 * kSlot <= 2 * G::kTile, "the slice's results fit the ring");
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  float* w = reinterpret_cast<float*>(smem + g * kSlot);
  if (slice == 1) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        reinterpret_cast<floatx4*>(w)[(db * 4 + r4) * 64 + lane] =
            floatx4{o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]};
    w[DB * 16 * 64 + lane] = m_run;
    w[DB * 16 * 64 + 64 + lane] = l_tot;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (slice == 1) return;
  {
    const float ms = w[DB * 16 * 64 + lane], ls = w[DB * 16 * 64 + 64 + lane];
    const float m_new = fmaxf(m_run, ms);
    const float f0 = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
    const float f1 = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - m_new);
    l_tot = l_tot * f0 + ls * f1;
    m_run = m_new;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const floatx4 x = reinterpret_cast<const floatx4*>(w)[(db * 4 + r4) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][4 * r4 + e] = o[db][4 * r4 + e] * f0 + x[e] * f1;
      }
  }
  // 0 times anything but a number is NaN
  float bad = l_tot * 0.f;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) bad = fmaf(o[db][r], 0.f, bad);
  if (pos < Lq && bad != 0.f) p.redo[wgi] = 1;
  if (pos >= Lq) return;
  l_tot *= kPerUnit;
  // register 4 r4 + e of block db: dimension 32 db + 8 r4 + 4 h + e
  if (p.splits > 1) {
    const int64_t prow = ((int64_t)split * (p.total / (p.splits * p.wgs_per_head)) + bhq) * Lq + pos;
    float* po = p.part_o + prow * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4)
        *reinterpret_cast<floatx4*>(po + 32 * db + 8 * r4 + 4 * h) =
            floatx4{o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]} * (kPerUnit * kPerUnit);
    if (h == 0) p.part_ml[prow] = make_float2(m_run, l_tot);
    return;
  }
  const float inv_l = l_tot > 0.f ? 1.0f / l_tot * (kPerUnit * kPerUnit) : 0.f;            // a row without any key: zeros
  float* op = reinterpret_cast<float*>(a.out) + a.out_offset(bhq, qrow);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *reinterpret_cast<floatx4*>(op + 32 * db + 8 * r4 + 4 * h) =
          floatx4{o[db][4 * r4], o[db][4 * r4 + 1], o[db][4 * r4 + 2], o[db][4 * r4 + 3]} * inv_l;
  if (a.lse && h == 0) a.lse[(int64_t)bhq * Lq + qrow] = lse_of(m_run, l_tot, p.lse_k);
}

// Adds up the partial results of the workgroups that shared a query's list: D/4 lanes per query.  The parts of kAtOnce workgroups are
// requested at once (past the last: the last again); one after the other their latencies were the kernel.
template <bool kBf16, int D, int kAtOnce>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnArgs a, const float* __restrict__ part_o,
                                                           const float2* __restrict__ part_ml, int splits, int64_t rows,
                                                           LseFactor lse_k) {
  constexpr int LPR = D / 4;
  const int64_t row = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;       // bhq * Lq + sorted position
  if (row >= rows) return;
  const int sub = threadIdx.x % LPR;
  const int Lq = a.q.L, bhq = (int)(row / Lq), pos = (int)(row - (int64_t)bhq * Lq);
  float2 ml[kAtOnce];
  floatx4 t[kAtOnce];
  auto request = [&](int s0) {
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      const int64_t at = min(s0 + j, splits - 1) * rows + row;
      ml[j] = part_ml[at];
      t[j] = *reinterpret_cast<const floatx4*>(part_o + at * D + 4 * sub);
    }
  };
  request(0);
  float m = -INFINITY, l = 0.f;
#pragma unroll
  for (int j = 0; j < kAtOnce; ++j) m = fmaxf(m, ml[j].x);
  for (int s = kAtOnce; s < splits; ++s) m = fmaxf(m, part_ml[s * rows + row].x);
  floatx4 o = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < splits; s0 += kAtOnce) {
    if (s0 > 0) request(s0);
#pragma unroll
    for (int j = 0; j < kAtOnce; ++j) {
      if (s0 + j >= splits || ml[j].y == 0.f) continue;    // nothing was seen there (and perhaps nothing written); not so a NaN
      const float f = __builtin_amdgcn_exp2f(ml[j].x - m);
      l = fmaf(ml[j].y, f, l);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(t[j][e], f, o[e]);
    }
  }
  const float inv_l = l > 0.f ? 1.0f / l : 0.f;
  const int qrow = perm_at(a.perm_q, (int64_t)bhq * Lq, pos, Lq);
  if constexpr (kBf16) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    bf16x4 t;
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] = (__bf16)(o[e] * inv_l);
    *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(a.out) + a.out_offset(bhq, qrow) + 4 * sub) = t;
  } else {
    *reinterpret_cast<floatx4*>(reinterpret_cast<float*>(a.out) + a.out_offset(bhq, qrow) + 4 * sub) = o * inv_l;
  }
  if (a.lse && sub == 0) a.lse[(int64_t)bhq * Lq + qrow] = lse_of(m, l, lse_k);
}

// How many workgroups share a list (`work` workgroups without splitting, QG x KS waves each): rounds of workgroups
// times (steps of one, a tile per slice each, plus its prologue and epilogue), plus the combining pass and its
// bytes.  The step times are measured (attn_f32_kernel at 1, 2 and 4 splits: 26.2, 17.0, 12.3 us for one head of
// L = 1024, d = B = 64, and 4.2 us for the combining pass; L = 4096, d = B = 128, 8 heads: 293 us unsplit, 315 + 11 in
// two).
struct Splits { int splits; double us; };
Splits plan_splits(int64_t work, int tiles, int KS, double step_us, size_t row_bytes, size_t ws_bytes) {
  Splits best{1, 0.0};
  for (int s = 1; s <= kMaxSplits && (s == 1 || (tiles >= s * KS && s * row_bytes <= ws_bytes)); ++s) {
    const double cost = (double)((work * s + kCUs - 1) / kCUs) * (ceil_div(tiles, s * KS) * step_us + 8.0) +
                        (s > 1 ? 4.0 + (double)(s * row_bytes) / 2e6 : 0.0);
    if (s == 1 || cost < best.us) best = Splits{s, cost};
  }
  return best;
}
double f32_step_us(int D, int waves) { return (D == 128 ? 9.2 : 4.5) * (waves == 8 ? 1.0 : 0.6); }
// Query groups and key slices of a workgroup: queries = the query block; slices so that its tiles fill the LDS (128 KB
// of ring).
struct F32Shape { int QG, KS; };
constexpr F32Shape shape_of(int d, int B) { return F32Shape{B / 32, d == 64 && B == 64 ? 4 : 2}; }

// One step of the three-part kernel, a 32-key tile per slice, at D = 64 and 128 (the chip full: 3.1 and 5.3 us; the longer
// of 24 and 12 MFMAs per 16 numbers and half of the softmax, twice).
constexpr double kSplitStepUs[2] = {3.2, 5.4};
size_t split_img_bytes(int BHkv, int Nk, int B, int d) { return align_up((size_t)BHkv * Nk * B * d * 12, 256); }
size_t split_redo_bytes(int BHq, int Nq, int B) { return align_up((size_t)BHq * ceil_div(Nq * B, 128) * 4, 256); }
constexpr size_t split_ring_bytes(int d) { return (size_t)2 * 12 * kTK * d; }      // a K and a V^T tile for each of two slices
size_t split_lds_bytes(int Nk, int d) { return split_ring_bytes(d) + (size_t)Nk * 4 + 8 * 4; }

// The three-part kernel or the other, for lists of `tiles` tiles and a workspace: the three-part one where its estimate,
// with the launches that go with it (9 us; 20 bytes per element of K and V at 5 TB/s), is the smaller one.  Attention call, fp32
// instruction -> this: 8 heads, L = 4096, keep 50 %, d = B = 128: 278 -> 182 us, d = 64: 149 -> 104; L = 6000: 645 -> 405 (two
// parts per list); 4 heads, L = 3001, keep 25 %: 69 -> 52; against, 2 heads, L = 1024: 30 / 31, L = 2048, B = 64: 40 / 47, d = B =
// 64, L = 2000: 24 / 30 at its best number of parts.
double three_part_fixed_us(size_t img) { return 9.0 + (double)img * 20.0 / 12.0 / 5e6; }
struct F32Plan { bool three_part; int splits; };
F32Plan plan_f32(int BHq, int BHkv, int Lq, int Lk, int d, int B, int tiles, bool causal, size_t ws_bytes) {
  const F32Shape f = shape_of(d, B);
  const int Nq = ceil_div(Lq, B), Nk = ceil_div(Lk, B);
  const size_t row_bytes = (size_t)BHq * Lq * (d * 4 + 8);
  const Splits plain = plan_splits((int64_t)BHq * ceil_div(Nq * B, 32 * f.QG), tiles, f.KS, f32_step_us(d, f.QG * f.KS), row_bytes,
                                   ws_bytes);
  const size_t img = split_img_bytes(BHkv, Nk, B, d), redo = split_redo_bytes(BHq, Nq, B);
  // (the membership words of the key blocks live in the ring while the list is built)
  if (causal || ws_bytes < img + redo || split_lds_bytes(Nk, d) > kLdsBytes || (size_t)Nk * 4 > split_ring_bytes(d))
    return F32Plan{false, plain.splits};
  const Splits three = plan_splits((int64_t)BHq * ceil_div(Nq * B, 128), B == 64 ? tiles + tiles / 12 : tiles, 2,
                                   kSplitStepUs[d == 128], row_bytes, ws_bytes - img - redo);
  const bool take = three.us + three_part_fixed_us(img) < plain.us;
  return F32Plan{take, take ? three.splits : plain.splits};
}

template <int D, int B>
basa_status launch_f32(F32Args p, int BHq, hipStream_t st) {
  constexpr int QG = shape_of(D, B).QG, KS = shape_of(D, B).KS;
  p.wgs_per_head = ceil_div(p.Nq * B, 32 * QG);
  const int work = BHq * p.wgs_per_head;                  // workgroups without splitting, one to a compute unit
  const int tiles = (p.a.row_cols ? std::min(p.a.cols_stride, p.Nk) : p.Nk) * (B / kTK);
  const int BHkv = p.a.k.batch * p.a.k.heads;
  const F32Plan plan = plan_f32(BHq, BHkv, p.a.q.L, p.a.k.L, D, B, tiles, p.a.causal != 0, p.a.ws_bytes);
  int splits = plan.splits;
  if (plan.three_part) {
    const size_t img = split_img_bytes(BHkv, p.Nk, B, D), redo = split_redo_bytes(BHq, p.Nq, B);
    const size_t lds_s = split_lds_bytes(p.Nk, D);
    static_assert(split_ring_bytes(D) == 2 * SplitGeo<D>::kTile, "a K and a V^T tile for each of two slices");
    SplitArgs s;
    s.wgs_per_head = ceil_div(p.Nq * B, 128);
    const int work_s = BHq * s.wgs_per_head;
    s.a = p.a; s.Nq = p.Nq; s.Nk = p.Nk; s.group = p.group; s.scale_log2e = p.scale_log2e; s.lse_k = p.lse_k;
    s.splits = plan.splits;
    s.total = work_s * s.splits;
    char* ws = reinterpret_cast<char*>(p.a.ws);
    s.img = ws;
    s.redo = reinterpret_cast<int32_t*>(ws + img);
    s.part_o = reinterpret_cast<float*>(ws + img + redo);
    s.part_ml = reinterpret_cast<float2*>(s.part_o + (size_t)s.splits * BHq * p.a.q.L * D);
    {
      ProfScope prof(K_GATHER, st);
      hipLaunchKernelGGL(split_kv_kernel<D>, dim3(p.Nk * (B / kTK), BHkv, 2), dim3(256), 0, st, p.a.k, p.a.v, p.a.perm_k, ws, s.redo,
                         work_s);
      BASA_HIP_CHECK_LAUNCH("split_kv_kernel");
    }
    {
      ProfScope prof(K_ATTN_F32, st);
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_split_kernel<D, B>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_s);
      if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");
      hipLaunchKernelGGL((attn_split_kernel<D, B>), dim3(s.total), dim3(512), lds_s, st, s);
      BASA_HIP_CHECK_LAUNCH("attn_split_kernel");
    }
    if (s.splits > 1) {
      const basa_status e = launch_attn_combine(p.a, s.part_o, s.part_ml, s.splits, st);
      if (e != BASA_OK) return e;
    }
    p.redo = s.redo;
    p.redo_wgs = s.wgs_per_head;
    splits = 1;                              // whole lists
  }
  p.splits = splits;
  p.total = work * splits;
  if (splits > 1) {
    p.part_o = reinterpret_cast<float*>(p.a.ws);
    p.part_ml = reinterpret_cast<float2*>(p.part_o + (size_t)splits * BHq * p.a.q.L * D);
  }
  const size_t lds = (size_t)KS * 2 * 2 * kTK * D * 4 + (p.a.causal ? KS * 2 * kTK * 4 : 0);
  {
    ProfScope prof(K_ATTN_F32, st);
#define BASA_F32(C, R)                                                                                           \
  do {                                                                                                           \
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_f32_kernel<D, QG, KS, C, R>),   \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(dynamic LDS)");                                 \
    hipLaunchKernelGGL((attn_f32_kernel<D, QG, KS, C, R>), dim3(p.total), dim3(64 * QG * KS), lds, st, p);       \
  } while (0)
    if (p.a.causal) BASA_F32(true, false);
    else if (p.redo) BASA_F32(false, true);
    else BASA_F32(false, false);
#undef BASA_F32
    BASA_HIP_CHECK_LAUNCH("attn_f32_kernel");
  }
  return splits > 1 ? launch_attn_combine(p.a, p.part_o, p.part_ml, splits, st) : BASA_OK;
}

}  // namespace

basa_status launch_attn_combine(const AttnArgs& a, const float* part_o, const float2* part_ml, int splits, hipStream_t st) {
  const int64_t rows = (int64_t)a.q.batch * a.q.heads * a.q.L;
  const int rpw = 256 / (a.q.d / 4);
  const dim3 grid((unsigned)((rows + rpw - 1) / rpw));
  ProfScope prof(K_ATTN_COMBINE, st);
  // Eight at once for two parts are six requests too many, which shows where there are many rows.  Combining pass, one part after the
  // other / eight at once / this rule: bf16, d = 128, two parts of 2 heads, L = 6500: 5.8 / 7.0 / 5.3 us, d = 64, 4 heads, L = 18350: 12.6 / 13.6 / 10.5; fp32, d =
  // 128, 2 heads, L = 6500: 6.3 / 7.6 / 5.9.
#define BASA_COMB_N(BF, D, N) \
  hipLaunchKernelGGL((attn_combine_kernel<BF, D, N>), grid, dim3(256), 0, st, a, part_o, part_ml, splits, rows, lse_factor(D))
#define BASA_COMB(BF, D)                          \
  do {                                            \
    if (splits <= 2) BASA_COMB_N(BF, D, 2);       \
    else if (splits <= 4) BASA_COMB_N(BF, D, 4);  \
    else BASA_COMB_N(BF, D, 8);                   \
  } while (0)
  const bool bf = a.q.dtype == BASA_BF16;
  if (bf && a.q.d == 128) BASA_COMB(true, 128);
  else if (bf) BASA_COMB(true, 64);
  else if (a.q.d == 128) BASA_COMB(false, 128);
  else BASA_COMB(false, 64);
#undef BASA_COMB
#undef BASA_COMB_N
  BASA_HIP_CHECK_LAUNCH("attn_combine_kernel");
  return BASA_OK;
}

// Room for the partial results of as many workgroups per list as could be of use (callers who hand over
// less get fewer): enough to give every compute unit two workgroups.  From two rounds of workgroups on, two parts per list
// help only where the last round is at most half full, and no room is asked for where they would not help lists of
// every block (or one less: an odd number splits worse); 32 heads of L = 131072 would ask for 4.4 GB.
size_t attn_f32_workspace_bytes(int BHq, int Lq, int Lk, int d, int B) {
  const int64_t wgs = (int64_t)BHq * ceil_div(Lq, 128);
  const size_t splits = (size_t)std::max<int64_t>(2, std::min<int64_t>(kMaxSplits, 2 * kCUs / wgs));
  const size_t row_bytes = (size_t)BHq * Lq * (d * 4 + 8);
  if (splits == 2) {
    const F32Shape f = shape_of(d, B);
    const int64_t work = (int64_t)BHq * ceil_div(Lq, 32 * f.QG);
    const int Nk = ceil_div(Lk, B);
    bool use = false;
    for (int n = std::max(1, Nk - 1); n <= Nk; ++n)
      use |= plan_splits(work, n * (B / kTK), f.KS, f32_step_us(d, f.QG * f.KS), row_bytes, 2 * row_bytes).splits > 1;
    if (!use) return 256;                                 // (non-zero for callers)
  }
  return align_up(splits * row_bytes, 256);
}
// With the tiles of the three-part kernel as well, and as many partial rows as lists of any length would have there, if lists
// of some length go to that kernel at all.
size_t attn_f32_best_workspace_bytes(int BHq, int BHkv, int Lq, int Lk, int d, int B, bool causal) {
  const size_t base = attn_f32_workspace_bytes(BHq, Lq, Lk, d, B);
  if (causal) return base;
  const int Nk = ceil_div(Lk, B);
  const size_t img = split_img_bytes(BHkv, Nk, B, d) + split_redo_bytes(BHq, ceil_div(Lq, B), B);
  const size_t row_bytes = (size_t)BHq * Lq * (d * 4 + 8);
  // (the other kernel with every block listed, already below what the three-part one takes with one tile: no length is for it)
  const F32Shape f = shape_of(d, B);
  if (plan_splits((int64_t)BHq * ceil_div(ceil_div(Lq, B) * B, 32 * f.QG), Nk * (B / kTK), f.KS, f32_step_us(d, f.QG * f.KS), row_bytes,
                  base).us < three_part_fixed_us(split_img_bytes(BHkv, Nk, B, d)) + 8.0 + kSplitStepUs[d == 128])
    return base;
  const int64_t work = (int64_t)BHq * ceil_div(Lq, 128);
  size_t splits = 0;            // (without what plan_f32 adds for two lists of 64: four heads, L = 3001, every block: 124 us, with
                                //  the parts that it would then take 128)
  for (int n = 1; n <= Nk; n += std::max(1, n / 8))
    splits = std::max<size_t>(splits, plan_splits(work, n * (B / kTK), 2, kSplitStepUs[d == 128], row_bytes, SIZE_MAX).splits);
  const size_t best = std::max(base, img + (splits > 1 ? align_up(splits * row_bytes, 256) : 0));
  for (int n = Nk; n >= 1; n -= std::max(1, n / 9))
    if (plan_f32(BHq, BHkv, Lq, Lk, d, B, n * (B / kTK), false, best).three_part) return best;
  return base;
}

basa_status launch_attn_f32(const AttnArgs& a, hipStream_t st) {
  const int BHq = a.q.batch * a.q.heads;
  F32Args p;
  p.a = a;
  p.Nq = ceil_div(a.q.L, a.B); p.Nk = ceil_div(a.k.L, a.B);
  if (BHq == 0 || p.Nq == 0) return BASA_OK;
  p.group = a.q.heads / a.k.heads;
  p.scale_log2e = 1.4426950408889634f / sqrtf((float)a.q.d);
  p.lse_k = lse_factor(a.q.d);
  p.part_o = nullptr; p.part_ml = nullptr; p.redo = nullptr; p.redo_wgs = 0;
  if (!a.ws || reinterpret_cast<uintptr_t>(a.ws) % 16) p.a.ws_bytes = 0;
  if (a.q.d == 128) return a.B == 128 ? launch_f32<128, 128>(p, BHq, st) : launch_f32<128, 64>(p, BHq, st);
  return a.B == 128 ? launch_f32<64, 128>(p, BHq, st) : launch_f32<64, 64>(p, BHq, st);
}

}  // namespace basa
