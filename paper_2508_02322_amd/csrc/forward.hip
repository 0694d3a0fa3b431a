// The layer output over the kept micro-experts (Eq. 1-2; the recomputed output
// of Algorithm 2, line 14) and its distance from the original output (the
// Lemma's decoding error; the L2 / cosine comparison of hidden states).
//
// The two contractions run in the grouped MFMA kernel (gemm.hip): first
// Lambda = a silu(X W_gate^T) (X W_up^T), masked and stored as bf16 per bucket
// slot, then Lambda W_down^T per slot in float32.  What is here:
//   combine : y_token (+)= the rows of its top-k slots, added in k order (a
//             token's experts are summed in a fixed order, no float atomics)
//   error   : per token ||y - y_hat||^2, ||y||^2, ||y_hat||^2, <y, y_hat>
#include "camera_internal.h"

namespace camera {
namespace {

constexpr int kThreads = 256;
constexpr int kTokensPerBlock = kThreads / kWave;  // one wave per token

// rows: product [pairs][d_model] float32.  Routed: slot_of[token * top_k + k]; dense: slot = e * n + token.
// grid: x = tokens, y = blockDim.x vectors of four columns each.  A workgroup has one token, so its slots are scalar
// loads, and the rows of eight terms are in flight together: waiting for each row in turn is what a wave per token
// spent its time on.  8192 tokens, 8 terms, 2048 wide: 143 -> 127 us; 2048 tokens, 2 terms, 4096 wide: 44 -> 19 us.
// PARTS: a slot's row is the sum of its rows of every part, in order; eight rows are in flight whatever terms and parts they are
// of.  An instance of its own: within the loop over terms the parts took 78 registers a lane where whole rows take 44, six waves
// per SIMD and not eight.  (STREAM needs no parts: rows that fill the cache are whole.)
constexpr int kTerms = 8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
template <bool STREAM, bool PARTS>
__global__ __launch_bounds__(kThreads) void combine_kernel(const f32x4* __restrict__ product,
                                                           const int32_t* __restrict__ slot_of, int64_t n, int top_k,
                                                           int n_experts, int vecs, int accumulate, int k_parts,
                                                           const int32_t* __restrict__ parts, int64_t part_stride,
                                                           f32x4* __restrict__ Y) {
  const int64_t tok = blockIdx.x;
  const int v = (int)(blockIdx.y * blockDim.x + threadIdx.x);
  const int terms = slot_of ? top_k : n_experts;
  if constexpr (!PARTS) {
    if (v >= vecs) return;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (accumulate) s = Y[tok * vecs + v];
    for (int k0 = 0; k0 < terms; k0 += kTerms) {
      int64_t row[kTerms];
      f32x4 p[kTerms];
#pragma unroll
      for (int u = 0; u < kTerms; ++u) {
        const int k = k0 + u;
        row[u] = k >= terms ? -1 : (slot_of ? (int64_t)slot_of[tok * top_k + k] : (int64_t)k * n + tok);
      }
#pragma unroll
      for (int u = 0; u < kTerms; ++u)
        if (row[u] >= 0)  // below 0: past the last term, or an expert id outside the group
          p[u] = STREAM ? __builtin_nontemporal_load(product + row[u] * vecs + v) : product[row[u] * vecs + v];
#pragma unroll
      for (int u = 0; u < kTerms; ++u) {
        if (row[u] >= 0) s += p[u];
      }
    }
    Y[tok * vecs + v] = s;
  } else {
    if (v >= vecs) return;
    if (parts != nullptr) k_parts = *parts;
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, term = s;
    if (accumulate) s = Y[tok * vecs + v];
    const f32x4* rows = product + v;  // of the part of the next row to load
    int k = 0, part = 0;              // the next row to load
    int part_add = 0;                 // part of the next row to add
    while (k < terms) {
      int64_t row[kTerms];
      f32x4 p[kTerms];
#pragma unroll
      for (int u = 0; u < kTerms; ++u) {
        row[u] = k >= terms ? -1 : (slot_of ? (int64_t)slot_of[tok * top_k + k] : (int64_t)k * n + tok);
        if (row[u] >= 0) p[u] = rows[row[u] * vecs];
        rows += part_stride;
        if (++part == k_parts) rows = product + v, part = 0, ++k;
      }
#pragma unroll
      for (int u = 0; u < kTerms; ++u) {
        if (row[u] >= 0) {
          term = part_add == 0 ? p[u] : term + p[u];
          if (part_add == k_parts - 1) s += term;
        }
        if (++part_add == k_parts) part_add = 0;
      }
    }
    Y[tok * vecs + v] = s;
  }
}

// A wave per token.  VEC: four columns per lane and load (rows of whole, aligned vectors), eight loads in flight; a column at
// a time waits for memory at every step: 2048 tokens of 4096 columns 32 -> 12.9 us, 1500 of 1024 9.9 -> 4.8.  From kVecColumns
// on: a wave of vectors is 256 columns, and loads past the end are made again of the last vector.  Graph replays, us, by
// columns / by vectors: 1500, 8192 and 50000 tokens of 64 columns 2.5 / 3.1, 4.0 / 4.6, 14.0 / 14.8, of 320 2.97 / 3.11,
// 4.90 / 4.93, 21.5 / 19.7, of 512 3.30 / 3.13, 5.75 / 5.28, 31.1 / 30.6.
constexpr int64_t kVecColumns = 512;
template <bool VEC>
__global__ __launch_bounds__(kThreads) void output_error_kernel(const float* __restrict__ Y,
                                                                const float* __restrict__ Y_hat, int64_t n,
                                                                int64_t d_model, int64_t ldy, int64_t ldh,
                                                                float* __restrict__ per_token) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t tok = (int64_t)linear_block() * kTokensPerBlock + wave;
  if (tok >= n) return;
  const float* y = Y + tok * ldy;
  const float* h = Y_hat + tok * ldh;
  float d2 = 0.f, yy = 0.f, hh = 0.f, yh = 0.f;
  auto add = [&](float a, float b) {
    const float d = a - b;
    d2 = fmaf(d, d, d2);
    yy = fmaf(a, a, yy);
    hh = fmaf(b, b, hh);
    yh = fmaf(a, b, yh);
  };
  if constexpr (VEC) {
    const f32x4* yv = reinterpret_cast<const f32x4*>(y);
    const f32x4* hv = reinterpret_cast<const f32x4*>(h);
    const int64_t vecs = d_model / 4;
    for (int64_t c0 = 0; c0 < vecs; c0 += 4 * kWave) {
      f32x4 a[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t c = c0 + u * kWave + lane, in = c < vecs ? c : vecs - 1;
        a[u] = yv[in];
        b[u] = hv[in];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (c0 + u * kWave + lane >= vecs) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) add(a[u][i], b[u][i]);
      }
    }
  } else {
    for (int64_t c = lane; c < d_model; c += kWave) add(y[c], h[c]);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    d2 += __shfl_xor(d2, m);
    yy += __shfl_xor(yy, m);
    hh += __shfl_xor(hh, m);
    yh += __shfl_xor(yh, m);
  }
  if (lane == 0) {
    per_token[tok * 4 + 0] = d2;
    per_token[tok * 4 + 1] = yy;
    per_token[tok * 4 + 2] = hh;
    per_token[tok * 4 + 3] = yh;
  }
}

}  // namespace

hipError_t launch_combine(hipStream_t stream, const float* product, const int32_t* slot_of, int64_t n, int top_k,
                          int n_experts, int64_t d_model, int accumulate, bool stream_product, int k_parts,
                          const int32_t* parts, int64_t part_stride, float* Y) {
  if (n <= 0) return hipSuccess;
  if (stream_product && k_parts > 1) return hipErrorInvalidValue;
  const int vecs = (int)(d_model / 4);
  const int threads = vecs < kThreads ? (vecs + kWave - 1) / kWave * kWave : kThreads;
  auto kern = stream_product ? combine_kernel<true, false> : k_parts > 1 ? combine_kernel<false, true> : combine_kernel<false, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)n, (unsigned)((vecs + threads - 1) / threads)), dim3(threads), 0,
                     stream, reinterpret_cast<const f32x4*>(product), slot_of, n, top_k, n_experts, vecs, accumulate,
                     k_parts, parts, part_stride / 4, reinterpret_cast<f32x4*>(Y));
  return hipGetLastError();
}

hipError_t launch_output_error(hipStream_t stream, const float* Y, const float* Y_hat, int64_t n, int64_t d_model,
                               int64_t ldy, int64_t ldh, float* per_token) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + kTokensPerBlock - 1) / kTokensPerBlock;
  const bool vec = d_model >= kVecColumns && (d_model | ldy | ldh) % 4 == 0 &&
                   (reinterpret_cast<uintptr_t>(Y) | reinterpret_cast<uintptr_t>(Y_hat)) % 16 == 0;
  hipLaunchKernelGGL(vec ? output_error_kernel<true> : output_error_kernel<false>, launch_grid(blocks), dim3(kThreads), 0, stream, Y, Y_hat, n, d_model, ldy,
                     ldh, per_token);
  return hipGetLastError();
}

}  // namespace camera
