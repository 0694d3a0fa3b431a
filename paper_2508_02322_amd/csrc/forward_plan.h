// The forms that the layer outputs take by their sizes, and the workspace for them.  It needs no HIP, so that a plain C++
// program can include it; what a kernel decides by the same rule is for the device too.
#pragma once

#include <stdint.h>

#include <algorithm>

#ifdef __HIPCC__
#define CAMERA_PLAN_FN __host__ __device__ inline
#else
#define CAMERA_PLAN_FN inline
#endif

namespace camera {

constexpr int kPlanCus = 256, kPlanDies = 8;     // compute units, on that many dies
constexpr int kPlanTileM = 256, kPlanTileN = 128, kPlanTileK = 64;  // the bf16 contraction's tile (gemm.hip): tokens, channels, K
constexpr int64_t kPlanCacheBytes = int64_t(256) << 20;  // the memory-side cache

// Whether the product rows of `pairs` slots go past the caches on their way out (second contraction) and back in
// (combine): from 256 MiB on, which is what the memory-side cache holds, they only displace each other in it.  Second
// contraction + combine, us, through the caches / past them: 537 MB 291 + 128 / 280 + 107 (8192 tokens of the DeepSeek
// shape, 40 % pruned), below the line 197 MB 338 + 106 / 335 + 114, 79 MB 74 + 30 / 70 + 35.
inline bool product_streams(int64_t pairs, int64_t d_model) { return pairs * d_model * 4 >= kPlanCacheBytes; }

// Column tiles of the second contraction: a tile takes its columns from both halves of d_model.
inline int64_t product_n_tiles(int64_t d_model) { return (d_model / 2 + kPlanTileN - 1) / kPlanTileN; }

// The most parts that a K extent is cut into: at least eight K tiles each.
constexpr int kMostParts = 8;
inline int most_k_parts(int64_t k_ext) {
  constexpr int kFewestTiles = 8;
  return (int)std::max<int64_t>(1, std::min<int64_t>(kMostParts, (k_ext + kPlanTileK - 1) / kPlanTileK / kFewestTiles));
}

// Time of the second contraction's `tiles` tiles (token tiles times column tiles) in parts of K, with the product rows that every
// part writes and the combine reads, in ns.  The tiles are dealt evenly to the dies, whose 32 units run them in rounds of 1.4 us
// per K tile and 8 us around them; a part's rows go at 6 TB/s while they fit the memory-side cache.  Whole numbers: host and device
// come to the same.
struct SplitCost {
  int64_t k_ns, part_ns;  // of all K tiles of a tile; of one part's rows
};
inline SplitCost split_cost(int64_t k_ext, int64_t product_bytes) {
  return {1400 * ((k_ext + kPlanTileK - 1) / kPlanTileK), 2 * product_bytes / 6000};
}
CAMERA_PLAN_FN int64_t tiles_per_die(int64_t tiles) { return (tiles + kPlanDies - 1) / kPlanDies; }
CAMERA_PLAN_FN int64_t split_ns(int64_t tiles, int parts, SplitCost c) {
  const int64_t rounds = (tiles_per_die(tiles) * parts + kPlanCus / kPlanDies - 1) / (kPlanCus / kPlanDies);
  return rounds * (c.k_ns / parts + 8000) + parts * c.part_ns;
}
// K is cut into the parts that take the shortest time, if that saves a sixth.  How many tiles there are depends on how the routed
// pairs fall on the experts, so the kernel decides (gemm.hip), by this rule: guessed from the number of pairs, the second
// contraction + combine of 1900 tokens of the Mixtral shape took four parts and 448 us where its 16 token tiles are one full
// round and 357, of 1150 tokens of 24 experts of 2048, 768 wide, three parts, 55 us, where two take 42.  Second contraction +
// combine, us, whole / in the parts taken: 2048 tokens of the Mixtral shape, 20 token tiles by 16 of 224 K tiles, 598 / 496;
// 300 and 2048 tokens of one expert of 20480, 3584 wide, 309 / 72 and 365 / 236; 500 tokens of 8 experts of 3072, 768 wide,
// 50 / 27.  Over 334 sizes of 20 shapes the parts taken are 0.8 % above the best and none is slower than whole (by a guess, and
// with rounds of all 256 units: 3.6 %, up to 1.26 times); a call that is left whole but might have been cut pays up to 4 % of these
// two kernels for the workgroups prepared for it.
CAMERA_PLAN_FN bool split_pays(int64_t ns, int64_t whole_ns) { return 100 * ns < 85 * whole_ns; }
inline int product_k_parts(int64_t tiles, int most, SplitCost c) {
  int best = 1;
  for (int p = 2; p <= most; ++p)
    if (split_ns(tiles, p, c) < split_ns(tiles, best, c)) best = p;
  return split_pays(split_ns(tiles, best, c), split_ns(tiles, 1, c)) ? best : 1;
}
// What a call with between least_m and most_m token tiles may come to: the most parts, and the workgroups (a multiple of the
// dies) that hold the tiles of every such number in the parts it takes.  A workgroup without a tile still waits for a compute
// unit's whole LDS (1.5 ns each at the end of the launch), so there are no more than that.
struct SplitPlan {
  int most_parts;
  int64_t blocks;
};
inline SplitPlan product_plan(int64_t least_m, int64_t most_m, int64_t d_model, int64_t k_ext, int64_t product_bytes) {
  const SplitCost c = split_cost(k_ext, product_bytes);
  const int64_t n_tiles = product_n_tiles(d_model), in_cache = (kPlanCacheBytes - 1) / std::max<int64_t>(1, product_bytes);
  const int most = (int)std::min<int64_t>(most_k_parts(k_ext), in_cache);
  SplitPlan plan{1, tiles_per_die(most_m * n_tiles) * kPlanDies};
  // from six rounds on no number of parts saves a sixth (they save less than one round)
  for (int64_t m = least_m; m <= most_m && m * n_tiles <= 6 * kPlanCus && most > 1; ++m) {
    const int p = product_k_parts(m * n_tiles, most, c);
    plan.most_parts = std::max(plan.most_parts, p);
    plan.blocks = std::max(plan.blocks, tiles_per_die(m * n_tiles) * p * kPlanDies);
  }
  return plan;
}
// The parts of a compacted layer's second contraction, of whose n_experts every token takes top_k (0: all of them) and the
// n_shared behind them.  Its tiles have as many K tiles as their expert keeps and are dealt to the dies by cost, and parts make
// them more even, so that a guess of their number and of rounds on all units serves better than the rule above: over 98 sizes of 8
// ragged layers 2.2 % above the best number of parts, none slower than whole.
inline int compact_k_parts(int64_t n, int64_t n_experts, int64_t top_k, int64_t n_shared, int64_t d_model, int64_t mean_kept) {
  const int64_t pairs = n * top_k, used = std::max<int64_t>(1, std::min(pairs, n_experts)), dense = (n + kPlanTileM - 1) / kPlanTileM;
  // one tile of each expert, or half a tile of each is padding
  const int64_t routed = top_k == 0 ? n_experts * dense : (pairs <= used * kPlanTileM ? used : pairs / kPlanTileM + used / 2);
  const int64_t tiles = (routed + n_shared * dense) * product_n_tiles(d_model);
  const int64_t product_bytes = n * ((top_k ? top_k : n_experts) + n_shared) * d_model * 4;
  const int64_t k_tiles = (mean_kept + kPlanTileK - 1) / kPlanTileK;
  auto us = [&](int parts) {
    const int64_t rounds = (tiles * parts + kPlanCus - 1) / kPlanCus;
    return rounds * (1.4 * (double)k_tiles / parts + 5.0) + 2.0 * parts * (double)product_bytes / 6e6;
  };
  int best = 1;
  for (int p = 2; p <= most_k_parts(mean_kept) && p * product_bytes < kPlanCacheBytes; ++p)
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

// When a masked call's first contraction is prepared to go over the list of the kept micro-experts: the list, the work table and the
// zeros are three launches before it (12-16 us where the list is not used, the zeros on top where it is), and a launch with few
// more tiles than compute units gains little from fewer.  Below the line a list won 4 us of 124 (2.5e10 products, 40 % pruned) or lost.
inline bool masks_by_list(int64_t n_pairs, int64_t d_model, int64_t d_ff) {
  return (double)n_pairs * d_model * d_ff >= 4e10;
}

// Whether the list pays, by what it leaves, which the device knows: tiles of the list and of everything, the K tiles of each, and the
// bytes of the hidden rows that are zeroed for it.  A die's units run its share of the tiles in rounds of 1.4 us per K tile and 8 us
// around them, 2.3 us more where columns are written one by one; zeros go at 7 TB/s.  First contraction with its preparations, us,
// everything computed as without a list / by list / as decided: 2048 tokens of the Mixtral shape, 2 % of the mask pruned 824 / 881 /
// 836, 20 % 820 / 711 / 704, 40 % 821 / 603 / 596; 4096 of the DeepSeek shape 5 % 300 / 354 / 305, 20 % 295 / 308 / 296, 40 % 293 /
// 247 / 241; 700 of the Qwen2 shape 5 % 438 / 462 / 448, 40 % 440 / 355 / 355; 600 of one expert of 20480 5 % 159 / 177 / 165, 60 %
// 153 / 97 / 97.
CAMERA_PLAN_FN bool list_pays(int64_t list_tiles, int64_t all_tiles, int64_t k_tiles, int64_t zero_bytes) {
  constexpr int kDieCus = kPlanCus / kPlanDies;
  const int64_t list_rounds = (tiles_per_die(list_tiles) + kDieCus - 1) / kDieCus, all_rounds = (tiles_per_die(all_tiles) + kDieCus - 1) / kDieCus;
  return list_rounds * (1400 * k_tiles + 10300) + zero_bytes / 7000 < all_rounds * (1400 * k_tiles + 8000);
}

}  // namespace camera
