// The layer outputs' plan by sizes, for the tests: plain C++ around the header the library is built from.
#include "../../paper_2508_02322_amd/csrc/forward_plan.h"

extern "C" {
// K parts of a second contraction with m_tiles token tiles for n_pairs rows; *most_parts and *blocks: what the call was planned
// for when it knew of between least_m and most_m
int product_k_parts(int64_t m_tiles, int64_t least_m, int64_t most_m, int64_t d_model, int64_t k_ext, int64_t n_pairs, int* most_parts,
                    int64_t* blocks) {
  const int64_t bytes = n_pairs * d_model * 4;
  const camera::SplitPlan plan = camera::product_plan(least_m, most_m, d_model, k_ext, bytes);
  *most_parts = plan.most_parts;
  *blocks = plan.blocks;
  return camera::product_k_parts(m_tiles * camera::product_n_tiles(d_model), plan.most_parts, camera::split_cost(k_ext, bytes));
}
int compact_k_parts(int64_t n, int64_t n_experts, int64_t top_k, int64_t n_shared, int64_t d_model, int64_t mean_kept) {
  return camera::compact_k_parts(n, n_experts, top_k, n_shared, d_model, mean_kept);
}
int64_t product_workspace(int64_t product_bytes, int64_t k_ext) { return camera::product_workspace(product_bytes, k_ext); }
int64_t compact_product_workspace(int64_t pairs, int64_t experts, int tiled, int64_t row_bytes, int64_t k_ext, int chunks) {
  return camera::compact_product_workspace(pairs, experts, tiled != 0, row_bytes, k_ext, chunks);
}
int compact_fills_tiles(int64_t pairs, int64_t experts) { return camera::compact_fills_tiles(pairs, experts); }
int product_streams(int64_t pairs, int64_t d_model) { return camera::product_streams(pairs, d_model); }
int list_pays(int64_t list_tiles, int64_t all_tiles, int64_t k_tiles, int64_t zero_bytes) {
  return camera::list_pays(list_tiles, all_tiles, k_tiles, zero_bytes);
}
int masks_by_list(int64_t pairs, int64_t d_model, int64_t d_ff) { return camera::masks_by_list(pairs, d_model, d_ff); }
}
