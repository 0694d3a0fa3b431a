// The forms that the layer outputs take by their sizes, and the workspace for them.  Host code that needs no HIP, so that a
// plain C++ program can include it.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace camera {

constexpr int kPlanCus = 256;                    // compute units
constexpr int kPlanTileM = 256, kPlanTileN = 128, kPlanTileK = 64;  // the bf16 contraction's tile (gemm.hip): tokens, channels, K
constexpr int64_t kPlanCacheBytes = int64_t(256) << 20;  // the memory-side cache

// Whether the product rows of `pairs` slots go past the caches on their way out (second contraction) and back in
// (combine): from 256 MiB on, which is what the memory-side cache holds, they only displace each other in it.  Second
// contraction + combine, us, through the caches / past them: 537 MB 291 + 128 / 280 + 107 (8192 tokens of the DeepSeek
// shape, 40 % pruned), below the line 197 MB 338 + 106 / 335 + 114, 79 MB 74 + 30 / 70 + 35.
inline bool product_streams(int64_t pairs, int64_t d_model) { return pairs * d_model * 4 >= kPlanCacheBytes; }

// About as many token tiles as `pairs` spread over n_experts make: one of each, or half a tile of each is padding.
inline int64_t expected_m_tiles(int64_t pairs, int64_t n_experts) {
  const int64_t used = std::max<int64_t>(1, std::min(pairs, n_experts));
  return pairs <= used * kPlanTileM ? used : pairs / kPlanTileM + used / 2;
}

// The most parts that a K extent is cut into: at least eight K tiles each.
inline int most_k_parts(int64_t k_ext) {
  constexpr int kMost = 8, kFewestTiles = 8;
  return (int)std::max<int64_t>(1, std::min<int64_t>(kMost, (k_ext + kPlanTileK - 1) / kPlanTileK / kFewestTiles));
}

// Into how many parts the K extent of the second contraction is cut when there are about `tiles` tiles: as many as make the
// 256 compute units' rounds of tiles (1.4 us per K tile of 64, 5 us around them) shortest with the product rows that every
// part writes and the combine reads (6 TB/s while they fit the memory-side cache), if that saves a sixth.  Second
// contraction, us, whole / in parts: 2048 tokens of the Mixtral shape, 320 tiles of 224 K tiles, 546 / 441 (and 9 -> 23 per
// combine); 500 tokens of 6 experts and a shared one of 8192, 72 tiles, 132 / 59; 300 tokens of 4 experts, 4096 wide, 64 tiles
// 63 / 40; 100 tokens, 8 experts of 4096 channels, 1024 wide, 36 / 16.
inline int product_k_parts(int64_t tiles, int64_t k_ext, int64_t product_bytes) {
  const int64_t k_tiles = (k_ext + kPlanTileK - 1) / kPlanTileK;
  auto us = [&](int parts) {
    const int64_t rounds = (tiles * parts + kPlanCus - 1) / kPlanCus;
    return rounds * (1.4 * (double)k_tiles / parts + 5.0) + 2.0 * parts * (double)product_bytes / 6e6;
  };
  int best = 1;
  for (int p = 2; p <= most_k_parts(k_ext) && p * product_bytes < kPlanCacheBytes; ++p)
    if (us(p) < us(best)) best = p;
  return us(best) < 0.85 * us(1) ? best : 1;
}

// Workspace for the product rows of a call (product_bytes: one part of them) and of every smaller batch of the same layer,
// which may take more parts: what a larger batch has made room for, no smaller one outgrows, so that after a call on the
// largest batch nothing is allocated, under graph capture included, and no captured graph loses the memory it names.
inline int64_t product_workspace(int64_t product_bytes, int64_t k_ext) {
  return std::max(product_bytes, std::min(most_k_parts(k_ext) * product_bytes, kPlanCacheBytes));
}

// Whether a compacted layer's batch runs on the tiled MFMA kernel and not on the streaming ones: from more than 64 tokens per
// expert on average.  kStreamingTokens: the most that a streaming batch has per expert, plus one.
constexpr int64_t kStreamingTokens = 65;
inline bool compact_fills_tiles(int64_t pairs, int64_t experts) { return pairs / experts >= kStreamingTokens; }
// Product rows of a compacted layer's call and of every smaller batch: parts of K on the tiled kernel, `chunks` of K on the
// streaming ones.  row_bytes: one product row.
inline int64_t compact_product_workspace(int64_t pairs, int64_t experts, bool tiled, int64_t row_bytes, int64_t k_ext, int chunks) {
  if (!tiled) return chunks * pairs * row_bytes;
  return std::max(product_workspace(pairs * row_bytes, k_ext), chunks * (kStreamingTokens * experts - 1) * row_bytes);
}

// When a masked call's first contraction goes over the list of the kept micro-experts: the lists, the zeros and the work table
// are three launches before it (25-33 us), and a launch with few more
// tiles than compute units gains little from fewer.  Masked call, first contraction + these, us, against computing every
// micro-expert and zeroing the pruned ones: 2.4e11 products of 40 % pruned 815 -> 575 + 32, of 20 % 808 -> 757 + 33, of nothing
// pruned 800 -> 805 + 21; 6.9e10 (40 %) 288 -> 212 + 29; 4.7e10 (60 %) 278 -> 155 + 20; below the line 2.5e10 (40 %) 124 -> 107 + 19,
// (20 %) 109 -> 112 + 20.
inline bool masks_by_list(int64_t n_pairs, int64_t d_model, int64_t d_ff) {
  return (double)n_pairs * d_model * d_ff >= 4e10;
}

}  // namespace camera
