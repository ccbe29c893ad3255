// Sizes of the bf16 attention kernels that follow from their shapes, the LDS of a workgroup above all.  Plain C++ without
// the device: what a launch asks for is checked on the host, for every list length.
#pragma once
#include <algorithm>
#include <cstddef>

namespace basa {

constexpr int kTileKeys = 64;
constexpr int kIxStride = kTileKeys + 4;    // causal: ints per tile of the key-index array (64 indices and 4 bounds, key_index_tile)
#ifndef BASA_ATTN_QR
#define BASA_ATTN_QR 7
#endif

// Sizes that follow from the head dimension D.
template <int D>
struct Geo {
  static constexpr int kRowBytes = D * 2;                    // one row of Q or K
  static constexpr int kChunksPerRow = kRowBytes / 16;       // 16-byte chunks per row: 16 or 8
  static constexpr int kTileBytes = kTileKeys * kRowBytes;   // one K tile; a V^T tile (D rows of 128 B) is as large
  static constexpr int kStageBytes = 2 * kTileBytes;         // K tile then V^T tile
  static constexpr int kKSteps = D / 16;                     // MFMA k-steps of S^T = K Q^T
  static constexpr int kDBlocks = D / 32;                    // 32-row blocks of O^T
  static constexpr int kChunksPerTile = kTileBytes / 1024;   // 1 KB direct-to-LDS loads per K (or V^T) tile
};
// Ring stages of a workgroup: one of 512 threads has the compute unit to itself and walks tiles in
// pairs (two slots of two); two workgroups of 256 threads share a compute unit and walk one by one.
// With 64 queries per wave: two, or, where the waves walk in spans (wide_spans), up to four (wide_stages).
// (Not with d = 64 or the causal mask, whose tiles are too short to hide the choice of the next one: 4527 -> 4721 us at
//  32 heads, L = 32768, d = 64; 2116 -> 2206 causal, L = 16384.  Nor with running maxima, where the compiler then sends the
//  accumulators through scratch.)
constexpr bool wide_spans(int d, bool causal, bool fast) { return d == 128 && !causal && fast; }
constexpr int stages_of(int threads, int qpw) { return threads == 512 && qpw == 32 ? 4 : 2; }
// k-steps of Q^T a wave of 64 queries keeps in registers (the rest is parked in LDS): all for D = 64
// (the causal variant of the 64-queries-per-wave kernel carries the two visibility limits and the
//  key indices of the half-tile on top: one more k-step of Q^T is parked)
// (the pass without running maxima needs no registers for them and keeps all of Q^T, 117.6-119.1 ms
//  against 119.7-120.5 with one k-step parked; its causal variant does better with two parked as before:
//  139-140 ms against 147 with one)
#ifndef BASA_ATTN_QR_FAST
#define BASA_ATTN_QR_FAST 8
#endif
constexpr int q_reg_steps(int d, int qpw, bool causal = false, bool fast = false) {
  return (qpw == 64 && d == 128) ? (fast && !causal ? BASA_ATTN_QR_FAST : BASA_ATTN_QR - (causal ? 1 : 0)) : d / 16;
}

template <int D>
size_t lds_bytes(int threads, int qpw, int Nk, bool causal = false, bool fast = false, int stages = 0) {
  const size_t park = (size_t)(threads / 64) * (qpw / 32) * (D / 16 - q_reg_steps(D, qpw, causal, fast)) * 1024;
  if (stages == 0) stages = stages_of(threads, qpw);
  const size_t base = (size_t)stages * Geo<D>::kStageBytes + park + (size_t)Nk * 4 + (threads / 64) * 4;
  return causal ? ((base + 15) & ~(size_t)15) + (size_t)stages * kIxStride * 4 : base;
}
// What a kernel without running maxima has of LDS besides (the words behind __syncthreads_or; read from its assembly).
constexpr size_t static_lds(bool fast) { return fast ? 256 : 0; }
// Ring stages of a 512-query workgroup that walks in spans and has its compute unit to itself: four, or what the list
// leaves room for.
constexpr size_t kLdsBytes = 160 * 1024;
template <int D>
int wide_stages(int Nk) {
  int s = 4;
  while (s > 2 && lds_bytes<D>(512, 64, Nk, false, true, s) + static_lds(true) > kLdsBytes) --s;
  return s;
}
// Ring stages of a launch.
template <int D>
int launch_stages(int threads, int qpw, int Nk, bool causal, bool fast) {
  return qpw == 64 && wide_spans(D, causal, fast) ? wide_stages<D>(Nk) : stages_of(threads, qpw);
}
// Key blocks whose membership words fit the smallest ring, where they live while a workgroup builds its union list.
template <int D>
constexpr size_t kMostBlocks = (size_t)2 * Geo<D>::kStageBytes / 4;
// The largest request, static words included, among the launches that a call of Nk key blocks may make.
template <int D>
size_t most_lds(int Nk) {
  size_t most = lds_bytes<D>(512, 32, Nk);
  for (const bool causal : {false, true})
    for (const bool fast : {false, true})
      most = std::max(most, lds_bytes<D>(512, 64, Nk, causal, fast, launch_stages<D>(512, 64, Nk, causal, fast)) + static_lds(fast));
  return std::max(most, lds_bytes<D>(256, 32, Nk, false, true) + static_lds(true));
}

}  // namespace basa
