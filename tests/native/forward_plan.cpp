// The layer outputs' plan by sizes, for the tests: plain C++ around the header the library is built from.
#include "../../paper_2508_02322_amd/csrc/forward_plan.h"

extern "C" {
int64_t expected_m_tiles(int64_t pairs, int64_t n_experts) { return camera::expected_m_tiles(pairs, n_experts); }
int product_k_parts(int64_t tiles, int64_t k_ext, int64_t product_bytes) { return camera::product_k_parts(tiles, k_ext, product_bytes); }
int64_t product_workspace(int64_t product_bytes, int64_t k_ext) { return camera::product_workspace(product_bytes, k_ext); }
int64_t compact_product_workspace(int64_t pairs, int64_t experts, int tiled, int64_t row_bytes, int64_t k_ext, int chunks) {
  return camera::compact_product_workspace(pairs, experts, tiled != 0, row_bytes, k_ext, chunks);
}
int compact_fills_tiles(int64_t pairs, int64_t experts) { return camera::compact_fills_tiles(pairs, experts); }
int product_streams(int64_t pairs, int64_t d_model) { return camera::product_streams(pairs, d_model); }
int masks_by_list(int64_t pairs, int64_t d_model, int64_t d_ff) { return camera::masks_by_list(pairs, d_model, d_ff); }
}
