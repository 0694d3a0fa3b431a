// A = Top&Norm(R X): router logits, softmax, top-k and renormalisation
// (Algorithm 1, line 2; the weights A_i(x) of Eq. 2).
//
// Logits L[j, e] = <x_j, R_e> (+ bias_e) are accumulated in float32: for bf16 on
// v_mfma_f32_16x16x32_bf16, for float32 with FMA and a wave reduction.  The
// logits of a block's tokens go through LDS so that eight lanes can walk the
// experts of one token: top_k rounds of "largest remaining logit, lower index on
// ties".
// The bits of a bf16 token's logits do not depend on the batch it is in, so
// neither does its choice of experts: both bf16 kernels add in one order, which
// follows from d_model alone.  Blocks of 32 K elements are dealt to four chains
// in turn; a chain adds its eight blocks of every range of 1024 elements one MFMA
// after the other, starting from zero, then its ranges in order; the logit is
// (((chain 0 + bias) + chain 1) + chain 2) + chain 3.
// Selection is on the logits (softmax is increasing, so this is the top-k of
// the probabilities); the kept weights are exp(L - max) over the softmax
// denominator, renormalised over the kept ones.
#include <hip/hip_bf16.h>

#include <type_traits>

#include "camera_internal.h"

namespace camera {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// f(integral_constant<int, LO>), ..., f(integral_constant<int, HI - 1>)
template <int LO, int HI, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (LO < HI) {
    f(std::integral_constant<int, LO>{});
    static_for<LO + 1, HI>(f);
  }
}

constexpr int kTokens = 32;  // tokens per block
constexpr int kSub = 8;      // lanes that share one token in the top-k stage
constexpr int kChains = 4;   // bf16: the order of additions, see above
constexpr int kBlockK = 32;
constexpr int kRangeBlocks = 32;
constexpr int kRangeK = kRangeBlocks * kBlockK;

// The value of another of the eight lanes that share a token (all or none of them active): after the steps 0, 1 and 2 every
// lane has met all eight.  0 and 1 are the lanes at distance 1 and 2; 2 is the mirror image in the eight, which will do
// for the distance 4 because the lanes of a quad agree by then.  (Data-parallel primitives: a few cycles, where a shuffle
// goes through the LDS crossbar.)
template <int STEP, class T>
__device__ __forceinline__ T lane_of_eight(T v) {
  constexpr int kCtrl = STEP == 0 ? 0xb1 : (STEP == 1 ? 0x4e : 0x141);  // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, true));
}

// Top-k of one token by kSub consecutive lanes: lane `sub` has experts sub, sub + kSub, ... of at most NE, read once into
// registers (a round that reads them from LDS again waits for each: with the other kernels of that time, graph replays of 8192
// tokens and 64 experts 24 -> 21 us, of one token and 256 experts 47 -> 34 us); each round takes the
// largest logit not yet taken (ties: lower index) and the lanes agree on it with three xor-shuffles.  s_row[0 .. n_experts)
// are the token's logits.  The lane `sub` keeps the weight of round `sub` until the denominator is known.
template <int NE>
__device__ __forceinline__ void topk_of_token(const float* s_row, int n_experts, int top_k, int renorm, int sub,
                                              int32_t* idx_out, float* w_out) {
  constexpr int kPer = NE / kSub;
  float v[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) v[i] = s_row[min(sub + i * kSub, n_experts - 1)];
  float row_max = -INFINITY;
#pragma unroll
  for (int i = 0; i < kPer; ++i) row_max = fmaxf(row_max, v[i]);  // a repeated last expert does not change it
  static_assert(kSub == 8, "lane_of_eight");
  static_for<0, 3>([&](auto step) { row_max = fmaxf(row_max, lane_of_eight<decltype(step)::value>(row_max)); });
  float denom = 0.0f;
  if (!renorm) {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (sub + i * kSub < n_experts) denom += __expf(v[i] - row_max);
#pragma unroll
    for (int m = kSub / 2; m >= 1; m >>= 1) denom += __shfl_xor(denom, m);
  }
  float prev_v = INFINITY;
  int prev_i = -1;
  float kept_sum = 0.0f, mine = 0.0f;
  for (int r = 0; r < top_k; ++r) {
    float best_v = -INFINITY;
    int best_i = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = sub + i * kSub;
      const bool not_taken = e < n_experts && (v[i] < prev_v || (v[i] == prev_v && e > prev_i));
      if (not_taken && (v[i] > best_v || (v[i] == best_v && e < best_i))) {
        best_v = v[i];
        best_i = e;
      }
    }
    static_for<0, 3>([&](auto step) {
      const float ov = lane_of_eight<decltype(step)::value>(best_v);
      const int oi = lane_of_eight<decltype(step)::value>(best_i);
      if (ov > best_v || (ov == best_v && oi < best_i)) {
        best_v = ov;
        best_i = oi;
      }
    });
    const float p = __expf(best_v - row_max);
    if (r < kSub) {
      if (sub == r) mine = p;
    } else if (sub == 0) {
      w_out[r] = p;
    }
    if (sub == 0) idx_out[r] = best_i;
    kept_sum += p;
    prev_v = best_v;
    prev_i = best_i;
  }
  const float inv = 1.0f / (renorm ? kept_sum : denom);
  if (sub < top_k) w_out[sub] = mine * inv;
  if (sub == 0)
    for (int r = kSub; r < top_k; ++r) w_out[r] *= inv;
}

// bf16: 32 tokens per block, NT tiles of 32 experts, K in chunks of four blocks, one for each chain, that go through LDS.
// The MFMA operand layout (lane = row, 8 consecutive K elements) makes neighbouring lanes read different rows, i.e.
// a different cache line per lane; fetched that way from global memory a wave instruction costs four times the
// address cycles of a coalesced one.  So the block fetches each chunk coalesced (a row's KC elements by KC / 8
// neighbouring threads, 16 bytes each), PF chunks ahead in registers (a block is alone on its CU for most sizes:
// what hides the latency of HBM is the number of its own loads in flight), stores it to LDS with rows padded by
// 16 bytes (conflict-free fragment reads), and four waves take the chunk's four blocks.  From two expert tiles on a second
// four waves take half of the experts: half the accumulators and running sums per wave, so that 128 experts fit 128
// registers and two workgroups a CU.  Against four waves that chained all of K (one accumulator, no ranges), us per call:
//   2048 wide, 64 experts:  2049 / 8192 / 65536 tokens 17.4 / 19.8 / 98 -> 16.5 / 19.3 / 96
//              128 experts: 2049 / 16384 / 65536       31 / 46 / 157 -> 30 / 43 / 157
//              256 experts: 2049 / 16384 / 65536       57 / 120 / 473 -> 50 / 110 / 433
// No load is conditional: a thread whose token, expert or K position lies outside reads a valid address all the
// same (row 0, or a page of zeros for the K tail); what it brings in is never used.  The chains of the
// waves are added through LDS in chain order.
template <int NT>
constexpr int kRouteThreads = NT == 1 ? 256 : 512;
template <int NT>
__global__ __launch_bounds__(kRouteThreads<NT>, NT == 4 ? 4 : 1) void route_bf16_kernel(const __hip_bfloat16* __restrict__ X, int64_t n,
                                                                       int d_model, int64_t ldx,
                                                                       const __hip_bfloat16* __restrict__ R, int64_t ldr,
                                                                       const float* __restrict__ bias, int n_experts,
                                                                       int top_k, int renorm,
                                                                       const __hip_bfloat16* __restrict__ zeros,
                                                                       int32_t* __restrict__ topk_idx,
                                                                       float* __restrict__ topk_w) {
  constexpr int kThreads = kRouteThreads<NT>;
  constexpr int KC = kChains * kBlockK;             // K elements per chunk
  constexpr int kRangeChunks = kRangeK / KC;
  constexpr int kRowB = KC * 2 + 16;                // bytes of a padded LDS row
  constexpr int kVecs = KC / 8;                     // 16-byte vectors per row
  constexpr int kRowsPerPass = kThreads / kVecs;    // rows the block fetches per pass
  constexpr int kXPasses = kTokens / kRowsPerPass;
  constexpr int kRPasses = NT * 32 / kRowsPerPass;
  constexpr int kParts = kThreads / (kChains * kWave);  // parts of the experts, a chain's waves take one each
  constexpr int TN = NT * 2 / kParts;               // tiles of 16 experts per wave
  constexpr int kTileBytes = (kTokens + NT * 32) * kRowB;
  constexpr int kLogitBytes = kTokens * (NT * 32 + 1) * 4;
  // the logits of the block's tokens lie over the chunk buffers: they are written after the last chunk was read
  __shared__ __align__(16) unsigned char s_raw[kTileBytes > kLogitBytes ? kTileBytes : kLogitBytes];
  unsigned char* s_x = s_raw;
  unsigned char* s_r = s_raw + kTokens * kRowB;
  float (*s_logit)[NT * 32 + 1] = reinterpret_cast<float (*)[NT * 32 + 1]>(s_raw);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int chain = wave % kChains, part = wave / kChains;
  const int row = lane % 16, quarter = lane / 16;
  const int64_t tok0 = (int64_t)linear_block() * kTokens;
  if (tok0 >= n) return;  // block-uniform: the last row of a large grid is longer than needed

  // fetch side: this thread's vector of every row it brings in
  const int vec = threadIdx.x % kVecs, row0 = threadIdx.x / kVecs;
  const __hip_bfloat16* x_src[kXPasses];
  const __hip_bfloat16* r_src[kRPasses];
#pragma unroll
  for (int p = 0; p < kXPasses; ++p) {
    const int64_t tok = tok0 + row0 + p * kRowsPerPass;
    x_src[p] = X + (tok < n ? tok : 0) * ldx + vec * 8;
  }
#pragma unroll
  for (int p = 0; p < kRPasses; ++p) {
    const int e = row0 + p * kRowsPerPass;
    r_src[p] = R + (int64_t)(e < n_experts ? e : 0) * ldr + vec * 8;
  }
  constexpr int PF = NT <= 2 ? 4 : 1;               // chunks in flight
  static_assert(kRangeChunks % PF == 0, "a range ends with the last slot");
  u32x4 xv[PF][kXPasses], rv[PF][kRPasses];
  auto fetch = [&](auto slot, int k0) {              // chunks past the end read the zero page
    constexpr int u = decltype(slot)::value;
    const bool k_ok = k0 + vec * 8 < d_model;        // d_model is a multiple of 8
#pragma unroll
    for (int p = 0; p < kXPasses; ++p) xv[u][p] = *reinterpret_cast<const u32x4*>(k_ok ? x_src[p] + k0 : zeros);
#pragma unroll
    for (int p = 0; p < kRPasses; ++p) rv[u][p] = *reinterpret_cast<const u32x4*>(k_ok ? r_src[p] + k0 : zeros);
  };
  auto stage = [&](auto slot) {
    constexpr int u = decltype(slot)::value;
#pragma unroll
    for (int p = 0; p < kXPasses; ++p)
      *reinterpret_cast<u32x4*>(s_x + (row0 + p * kRowsPerPass) * kRowB + vec * 16) = xv[u][p];
#pragma unroll
    for (int p = 0; p < kRPasses; ++p)
      *reinterpret_cast<u32x4*>(s_r + (row0 + p * kRowsPerPass) * kRowB + vec * 16) = rv[u][p];
  };

  f32x4 acc[2][TN], sum[2][TN];  // of 2 x 16 tokens: the range that runs, the ranges before it
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < TN; ++t) acc[m][t] = sum[m][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  auto end_range = [&] {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        sum[m][t] += acc[m][t];
        acc[m][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      }
  };

  const int n_chunks = (d_model + KC - 1) / KC;
  const int col = (chain * kBlockK + quarter * 8) * 2;  // byte column of this lane's K elements
  static_for<0, PF>([&](auto u) { fetch(u, decltype(u)::value * KC); });
  for (int c0 = 0; c0 < n_chunks; c0 += PF) {
    static_for<0, PF>([&](auto u) {
      const int c = c0 + decltype(u)::value;
      if (c < n_chunks) {  // block-uniform
        stage(u);          // waits for this slot's loads only: the younger chunks stay in flight
        __syncthreads();
        fetch(u, (c + PF) * KC);
        bf16x8 a[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) a[m] = *reinterpret_cast<const bf16x8*>(s_x + (m * 16 + row) * kRowB + col);
#pragma unroll
        for (int t = 0; t < TN; ++t) {
          const bf16x8 b = *reinterpret_cast<const bf16x8*>(s_r + ((part * TN + t) * 16 + row) * kRowB + col);
#pragma unroll
          for (int m = 0; m < 2; ++m) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b, acc[m][t], 0, 0, 0);
        }
        if (decltype(u)::value == PF - 1 && (c + 1) % kRangeChunks == 0) end_range();  // block-uniform
        __syncthreads();  // every wave has read the chunk (after the last one: the logits may overwrite it)
      }
    });
  }
  if (n_chunks % kRangeChunks != 0) end_range();
  // accumulator element i of a lane: token 4 * quarter + i, expert `row` of the tile
  for (int w = 0; w < kChains; ++w) {  // fixed order: chain 0 stores (with the bias), chains 1..3 add
    if (chain == w) {
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int e = (part * TN + t) * 16 + row;
        const float b = (w == 0 && bias && e < n_experts) ? bias[e] : 0.0f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float* dst = &s_logit[m * 16 + 4 * quarter + i][e];
            *dst = (w == 0 ? 0.0f : *dst) + sum[m][t][i] + b;
          }
      }
    }
    __syncthreads();
  }
  const int t_local = threadIdx.x / kSub, sub = threadIdx.x % kSub;  // 256 threads = 32 tokens x 8 lanes
  if (t_local < kTokens && tok0 + t_local < n)
    topk_of_token<NT * 32>(s_logit[t_local], n_experts, top_k, renorm, sub, topk_idx + (tok0 + t_local) * top_k,
                     topk_w + (tok0 + t_local) * top_k);
}

// bf16, few tokens: a block per 32 tokens is one or two workgroups for a decoding batch, which fetch the whole router matrix
// in a sequence of chunks, a latency each.  So the ranges of K go to workgroups of their own, and so do groups of ET tiles of
// 16 experts (blockIdx.z): 16 tokens each, a wave per chain, its eight blocks straight from memory into the operands of
// v_mfma_f32_16x16x32_bf16 (the four lanes of a row read a 64-byte sector).  part [range][chain][n][n_experts] goes to memory
// as it is and route_pick_kernel adds it up.
constexpr int kTokensSmall = 16;
template <int ET>
__global__ __launch_bounds__(kWave * kChains) void route_bf16_split_kernel(
    const __hip_bfloat16* __restrict__ X, int64_t n, int d_model, int64_t ldx, const __hip_bfloat16* __restrict__ R,
    int64_t ldr, int n_experts, const __hip_bfloat16* __restrict__ zeros, float* __restrict__ part) {
  constexpr int kBlocks = kRangeBlocks / kChains;  // of a wave, all in flight
  const int lane = threadIdx.x % kWave, chain = threadIdx.x / kWave;
  const int row = lane % 16, quarter = lane / 16;
  const int64_t tok0 = (int64_t)blockIdx.x * kTokensSmall;
  const int e0 = blockIdx.z * ET * 16 + row;
  const __hip_bfloat16* x = X + min(tok0 + row, n - 1) * ldx;  // rows outside repeat the last one; never used
  const __hip_bfloat16* r[ET];
#pragma unroll
  for (int t = 0; t < ET; ++t) r[t] = R + (int64_t)min(e0 + t * 16, n_experts - 1) * ldr;
  f32x4 acc[ET];
#pragma unroll
  for (int t = 0; t < ET; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  bf16x8 xv[kBlocks], rv[kBlocks][ET];
#pragma unroll
  for (int u = 0; u < kBlocks; ++u) {
    const int k = ((int)blockIdx.y * kRangeBlocks + u * kChains + chain) * kBlockK + quarter * 8;
    const bool k_ok = k < d_model;  // d_model is a multiple of 8
    xv[u] = *reinterpret_cast<const bf16x8*>(k_ok ? x + k : zeros);
#pragma unroll
    for (int t = 0; t < ET; ++t) rv[u][t] = *reinterpret_cast<const bf16x8*>(k_ok ? r[t] + k : zeros);
  }
#pragma unroll
  for (int u = 0; u < kBlocks; ++u)
#pragma unroll
    for (int t = 0; t < ET; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv[u], rv[u][t], acc[t], 0, 0, 0);
  // accumulator element i of a lane: token 4 * quarter + i, expert `row` of the tile
  float* out = part + ((int64_t)blockIdx.y * kChains + chain) * n * n_experts;
#pragma unroll
  for (int t = 0; t < ET; ++t) {
    const int e = e0 + t * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t tok = tok0 + 4 * quarter + i;
      if (tok < n && e < n_experts) out[tok * n_experts + e] = acc[t][i];
    }
  }
}

// part [ranges][kChains][n][n_experts].  A thread has one logit, a block 256 / NE tokens, so that what it reads is one round
// of loads.  A thread counts the logits of its token that come before its own (larger, or equal with a lower index): that is
// its place in the top-k, without rounds that wait for each other.  The weights are those of topk_of_token bit for bit: the
// same exponentials, added in the same order.  (8 tokens per block and their top-k in rounds, against this, us, top 8 or 6:
// 1 token of 64 experts 7.9 / 5.2, 64 of 64 11.2 / 5.8, 16 of 128 18.3 / 8.5, 397 of 128 19.2 / 8.9, 250 of 256 (top 4) 20.8 / 15.0.)
template <int NE>
constexpr int kTokensPick = 256 / NE;
template <int NE>
__global__ __launch_bounds__(256) void route_pick_kernel(const float* __restrict__ part, int ranges, int64_t n,
                                                         const float* __restrict__ bias, int n_experts, int top_k,
                                                         int renorm, int32_t* __restrict__ topk_idx,
                                                         float* __restrict__ topk_w) {
  constexpr int T = kTokensPick<NE>;
  __shared__ __align__(16) float s_logit[T][NE + 4];
  __shared__ float s_v[T][NE], s_p[T][NE];  // logits by place, then their exponentials
  __shared__ int s_i[T][NE];
  const int t = threadIdx.x / NE, e = threadIdx.x % NE;
  const int64_t tok = (int64_t)blockIdx.x * T + t;
  const bool valid = tok < n && e < n_experts;
  float logit = __builtin_nanf("");  // of no expert: comes before none
  if (valid) {
    const int64_t stride = n * n_experts;
    const float* p = part + tok * n_experts + e;
    float sum[kChains] = {};
    for (int s0 = 0; s0 < ranges; s0 += 4) {  // the chains of four ranges in flight, added in range order
      float v[4][kChains];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < kChains; ++w) v[u][w] = p[(min(s0 + u, ranges - 1) * kChains + w) * stride];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int w = 0; w < kChains; ++w)
          if (s0 + u < ranges) sum[w] += v[u][w];
    }
    logit = sum[0] + (bias ? bias[e] : 0.0f);
#pragma unroll
    for (int w = 1; w < kChains; ++w) logit += sum[w];
  }
  s_logit[t][e] = logit;
  s_v[t][e] = -INFINITY;  // what a place holds that no logit takes (a token with NaN logits)
  s_i[t][e] = 0x7fffffff;
  __syncthreads();
  if (valid && logit == logit) {
    int place = 0;
#pragma unroll 8
    for (int j = 0; j < NE; j += 4) {
      const f32x4 o = *reinterpret_cast<const f32x4*>(&s_logit[t][j]);
#pragma unroll
      for (int u = 0; u < 4; ++u) place += (o[u] > logit || (o[u] == logit && j + u < e)) ? 1 : 0;
    }
    if (place < top_k) {
      s_v[t][place] = logit;
      s_i[t][place] = e;
    }
  }
  __syncthreads();
  const float row_max = s_v[t][0];
  const float kept = __expf(s_v[t][e] - row_max);  // of place e
  s_p[t][e] = renorm ? kept : __expf(logit - row_max);
  __syncthreads();
  if (tok >= n || e >= top_k) return;
  float total = 0.0f;
  if (renorm) {
    for (int r = 0; r < top_k; ++r) total += s_p[t][r];
  } else {  // the sums of kSub lanes that take every kSub-th expert, then these at distances 4, 2, 1
    float sub[kSub];
#pragma unroll
    for (int q = 0; q < kSub; ++q) {
      sub[q] = 0.0f;
      for (int i = q; i < n_experts; i += kSub) sub[q] += s_p[t][i];
    }
    total = ((sub[0] + sub[4]) + (sub[2] + sub[6])) + ((sub[1] + sub[5]) + (sub[3] + sub[7]));
  }
  topk_idx[tok * top_k + e] = s_i[t][e];
  topk_w[tok * top_k + e] = kept * (1.0f / total);
}

// float32: 8 tokens per block; its four waves deal the experts among them, EG at a time.  A wave's lanes stride over
// d_model with 8 x EG partial dot products in registers, so a row of R fetched once serves 8 tokens and a token fetched
// once EG experts.  What bounds it is the latency of one wave's loads, so blocks are small: 512 tokens are 64 of them.
// The partials of the 64 lanes are added by halving: at distance m a lane hands over half of its sums and keeps the
// other half, 8 * EG shuffles in all instead of 6 for each sum.  The order of the additions is a lane's K positions in
// turn and then lane distances 32, 16, ... 1: one float32 chain of d_model / 64 terms and a tree, which matters for ties.
// One token by one expert at a time and 32 tokens per block, as it was before, against this:
//   512 tokens, 8 experts, 256 wide     26 -> 4.9 us
//   1499 tokens, 12 experts, 772 wide   79 -> 9.9 us
constexpr int kTokensF32 = 8;
template <int EG, int NE>
__global__ __launch_bounds__(256) void route_f32_kernel(const float* __restrict__ X, int64_t n, int d_model,
                                                        int64_t ldx, const float* __restrict__ R, int64_t ldr,
                                                        const float* __restrict__ bias, int n_experts, int top_k,
                                                        int renorm, int32_t* __restrict__ topk_idx,
                                                        float* __restrict__ topk_w) {
  __shared__ float s_logit[kTokensF32][NE + 1];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t tok0 = (int64_t)linear_block() * kTokensF32;
  if (tok0 >= n) return;  // block-uniform: the last row of a large grid is longer than needed
  const float* x[kTokensF32];
#pragma unroll
  for (int t = 0; t < kTokensF32; ++t) x[t] = X + min(tok0 + t, n - 1) * ldx;  // tokens past the end repeat the last one
  for (int e0 = wave * EG; e0 < n_experts; e0 += 4 * EG) {
    const float* r[EG];
#pragma unroll
    for (int j = 0; j < EG; ++j) r[j] = R + (int64_t)min(e0 + j, n_experts - 1) * ldr;
    float s[kTokensF32 * EG];
#pragma unroll
    for (int i = 0; i < kTokensF32 * EG; ++i) s[i] = 0.0f;
#pragma unroll 2
    for (int c = lane * 4; c < d_model; c += kWave * 4) {  // d_model is a multiple of 4
      float4 rv[EG];
#pragma unroll
      for (int j = 0; j < EG; ++j) rv[j] = *reinterpret_cast<const float4*>(r[j] + c);
#pragma unroll
      for (int t = 0; t < kTokensF32; ++t) {
        const float4 xv = *reinterpret_cast<const float4*>(x[t] + c);
#pragma unroll
        for (int j = 0; j < EG; ++j) {
          float v = s[t * EG + j];
          v = fmaf(xv.x, rv[j].x, v);
          v = fmaf(xv.y, rv[j].y, v);
          v = fmaf(xv.z, rv[j].z, v);
          s[t * EG + j] = fmaf(xv.w, rv[j].w, v);
        }
      }
    }
    // After the step at distance m a lane holds the sums whose index has the lane's bit m in the place of that step.
    int held = 0;  // index of the one sum the lane ends with
    static_for<0, 6>([&](auto step) {
      constexpr int k = decltype(step)::value;
      constexpr int m = 32 >> k;
      constexpr int half = (kTokensF32 * EG) >> (k + 1);
      if constexpr (half >= 1) {
        const bool high = (lane & m) != 0;
        held += high ? half : 0;
#pragma unroll
        for (int i = 0; i < half; ++i) {
          const float keep = high ? s[i + half] : s[i];
          const float give = high ? s[i] : s[i + half];
          s[i] = keep + __shfl_xor(give, m);
        }
      } else {
        s[0] += __shfl_xor(s[0], m);
      }
    });
    constexpr int kCopies = kWave / (kTokensF32 * EG);  // lanes that end with the same sum
    const int t = held / EG, e = e0 + held % EG;
    if (lane % kCopies == 0 && e < n_experts) s_logit[t][e] = s[0] + (bias ? bias[e] : 0.0f);
  }
  __syncthreads();
  const int t_local = threadIdx.x / kSub, sub = threadIdx.x % kSub;  // one wave = 8 tokens x 8 lanes
  if (t_local < kTokensF32 && tok0 + t_local < n)
    topk_of_token<NE>(s_logit[t_local], n_experts, top_k, renorm, sub, topk_idx + (tok0 + t_local) * top_k,
                     topk_w + (tok0 + t_local) * top_k);
}

template <int NT>
void launch_bf16(hipStream_t stream, int64_t n_blocks, const void* X, int64_t n, int64_t d_model, int64_t ldx,
                 const void* W_r, int64_t ldr, const float* bias, int n_experts, int top_k, int renorm,
                 const void* zeros, int32_t* topk_idx, float* topk_w) {
  hipLaunchKernelGGL(route_bf16_kernel<NT>, launch_grid(n_blocks), dim3(kRouteThreads<NT>), 0, stream,
                     static_cast<const __hip_bfloat16*>(X), n, (int)d_model, ldx,
                     static_cast<const __hip_bfloat16*>(W_r), ldr, bias, n_experts, top_k, renorm,
                     static_cast<const __hip_bfloat16*>(zeros), topk_idx, topk_w);
}

// Whether a call goes range by range, then: it needs two ranges, room for their partial logits, and few enough tokens.  The
// block kernel's time hardly depends on the batch below 8192 tokens; that of the two launches grows with what they hand
// over, 16 bytes per logit and range.  us per call, block kernel / range by range:
//   8 experts, 4096 wide:     1 token 13.2 / 5.3,  1024 15.0 / 7.2,  4096 16.7 / 12.7
//   64 experts, 2048 wide:    1 token 15.3 / 11.7, 1024 16.4 / 14.5, 2048 16.5 / 18.8
//   128 experts, 2048 wide:   1 token 26.5 / 20.0, 1024 29.5 / 28.0, 2048 29.8 / 34.6
//   256 experts, 2048 wide:   1 token 46 / 31,     1024 49.1 / 49.2, 2048 49 / 59
// so the line is at 1024 tokens from 64 experts on, and below that where as many logits are, in whole tiles of 16 experts.
constexpr int64_t kSplitLogits = 1024 * 64;
bool route_split(int64_t n, int64_t ranges, int n_experts) {
  const int64_t experts = n_experts < 16 ? 16 : (n_experts > 64 ? 64 : n_experts);
  return ranges > 1 && n * experts <= kSplitLogits &&
         ranges * kChains * n * n_experts * (int64_t)sizeof(float) <= (int64_t)kRouteScratchBytes;
}

template <int NE>
void launch_bf16_split(hipStream_t stream, const void* X, int64_t n, int64_t d_model, int64_t ldx, const void* W_r,
                       int64_t ldr, const float* bias, int n_experts, int top_k, int renorm, const void* zeros,
                       float* scratch, int32_t* topk_idx, float* topk_w) {
  constexpr int ET = NE <= 16 ? 1 : 2;
  const int ranges = (int)((d_model + kRangeK - 1) / kRangeK);
  hipLaunchKernelGGL(route_bf16_split_kernel<ET>, dim3((unsigned)((n + kTokensSmall - 1) / kTokensSmall), (unsigned)ranges,
                     (unsigned)((n_experts + ET * 16 - 1) / (ET * 16))), dim3(kWave * kChains), 0, stream,
                     static_cast<const __hip_bfloat16*>(X), n, (int)d_model, ldx, static_cast<const __hip_bfloat16*>(W_r), ldr,
                     n_experts, static_cast<const __hip_bfloat16*>(zeros), scratch);
  hipLaunchKernelGGL(route_pick_kernel<NE>, dim3((unsigned)((n + kTokensPick<NE> - 1) / kTokensPick<NE>)), dim3(256), 0, stream, scratch,
                     ranges, n, bias, n_experts, top_k, renorm, topk_idx, topk_w);
}

}  // namespace

hipError_t launch_route_topk(hipStream_t stream, const void* X, int dtype, int64_t n, int64_t d_model,
                             int64_t ldx, const void* W_r, int64_t ldr, const float* bias, int n_experts,
                             int top_k, int renorm, const void* zeros, float* scratch, int32_t* topk_idx,
                             float* topk_w) {
  if (n <= 0) return hipSuccess;
  const int64_t n_blocks = (n + kTokens - 1) / kTokens;
  if (dtype == CAMERA_BF16) {
    if (route_split(n, (d_model + kRangeK - 1) / kRangeK, n_experts)) {
#define CAMERA_ROUTE_SPLIT(NE)                                                                                          \
  launch_bf16_split<NE>(stream, X, n, d_model, ldx, W_r, ldr, bias, n_experts, top_k, renorm, zeros, scratch, topk_idx, \
                        topk_w)
      if (n_experts <= 16) CAMERA_ROUTE_SPLIT(16);
      else if (n_experts <= 64) CAMERA_ROUTE_SPLIT(64);
      else if (n_experts <= 128) CAMERA_ROUTE_SPLIT(128);
      else CAMERA_ROUTE_SPLIT(256);
#undef CAMERA_ROUTE_SPLIT
      return hipGetLastError();
    }
    const int nt = (n_experts + 31) / 32;
#define CAMERA_ROUTE_CASE(NT)                                                                                        \
  launch_bf16<NT>(stream, n_blocks, X, n, d_model, ldx, W_r, ldr, bias, n_experts, top_k, renorm, zeros, topk_idx, \
                  topk_w)
    if (nt <= 1) CAMERA_ROUTE_CASE(1);
    else if (nt <= 2) CAMERA_ROUTE_CASE(2);
    else if (nt <= 4) CAMERA_ROUTE_CASE(4);
    else CAMERA_ROUTE_CASE(8);
#undef CAMERA_ROUTE_CASE
  } else {
    // two experts at a time where that is what keeps all four waves busy (up to 8 experts), four beyond
    auto kern = n_experts <= 8     ? route_f32_kernel<2, 8>
                : n_experts <= 64  ? route_f32_kernel<4, 64>
                : n_experts <= 128 ? route_f32_kernel<4, 128>
                                   : route_f32_kernel<4, CAMERA_MAX_EXPERTS>;
    hipLaunchKernelGGL(kern, launch_grid((n + kTokensF32 - 1) / kTokensF32), dim3(256), 0, stream,
                       static_cast<const float*>(X), n, (int)d_model, ldx, static_cast<const float*>(W_r), ldr,
                       bias, n_experts, top_k, renorm, topk_idx, topk_w);
  }
  return hipGetLastError();
}

}  // namespace camera
