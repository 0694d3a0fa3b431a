// Token -> expert bucketing: a stable counting sort of the n*top_k routed
// (token, expert) pairs by expert.  This is the explicit form of the masking
// by A[:, i] in Algorithm 1, line 6: expert i only ever sees the tokens whose
// routing weight to it is non-zero.
//
// Three launches, all integer work:
//   count   : every block histograms its 1024 consecutive pairs (LDS atomics)
//   scan    : one block turns the per-block histograms into exclusive bases,
//             and builds counts / offsets / the M-tile tables of the GEMM
//   scatter : every wave walks its 256 consecutive pairs 64 at a time; the
//             position of a pair inside its expert is found with wavefront
//             ballots (one per bit of the expert id gives the lanes of equal
//             expert) and popcounts of the lower lanes, so equal experts keep
//             their pair order (stable, deterministic).
// For few pairs one workgroup does all of it in one launch (bucket_small_kernel).
#include "camera_internal.h"

namespace camera {
namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;
constexpr int kPairsPerWave = kBucketChunk / kWavesPerBlock;  // 256
static_assert(kPairsPerWave % kWave == 0, "wave chunk must be whole wavefronts");

__global__ __launch_bounds__(kThreads) void bucket_count_kernel(const int32_t* __restrict__ topk_idx,
                                                                int64_t n_pairs, int n_experts,
                                                                int32_t* __restrict__ block_hist) {
  __shared__ int32_t hist[CAMERA_MAX_EXPERTS];
  for (int e = threadIdx.x; e < n_experts; e += kThreads) hist[e] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kBucketChunk;
  for (int i = threadIdx.x; i < kBucketChunk; i += kThreads) {
    const int64_t p = base + i;
    if (p < n_pairs) {
      const int e = topk_idx[p];
      if (e >= 0 && e < n_experts) atomicAdd(&hist[e], 1);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < n_experts; e += kThreads)
    block_hist[(int64_t)blockIdx.x * n_experts + e] = hist[e];
}

// One block.  Four threads per expert (neighbours), each with a quarter of the blocks: it sums its quarter, takes the sums
// of the quarters before it and the expert prefix from shuffles, and writes the exclusive bases in a second walk.  A lone
// workgroup is bound by the latency of its loads: eight at a time, and a quarter of the chain that one thread per expert
// would be (128 blocks x 128 experts: 18.5 -> 10 us; 64 x 64: 8.4 -> 4.6 us).
constexpr int kQuarters = 4;
constexpr int kScanThreads = CAMERA_MAX_EXPERTS * kQuarters;
static_assert(kScanThreads <= 1024, "one workgroup");
__global__ __launch_bounds__(kScanThreads) void bucket_scan_kernel(int32_t* __restrict__ block_hist, int n_blocks,
                                                                   int n_experts, int tile_m, int max_tiles,
                                                                   int32_t* __restrict__ counts,
                                                                   int32_t* __restrict__ offsets,
                                                                   int32_t* __restrict__ tile_offset,
                                                                   int32_t* __restrict__ tile_expert) {
  __shared__ int32_t s_pairs[kScanThreads / kWave], s_tiles[kScanThreads / kWave];
  const int e = threadIdx.x / kQuarters, quarter = threadIdx.x % kQuarters;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int b_begin = (int)((int64_t)n_blocks * quarter / kQuarters), b_end = (int)((int64_t)n_blocks * (quarter + 1) / kQuarters);
  const bool live = e < n_experts;
  int32_t* column = block_hist + e;
  int32_t mine = 0;
  if (live) {
    int b = b_begin;
    for (; b + 8 <= b_end; b += 8) {
      int32_t c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = column[(int64_t)(b + u) * n_experts];
#pragma unroll
      for (int u = 0; u < 8; ++u) mine += c[u];
    }
    for (; b < b_end; ++b) mine += column[(int64_t)b * n_experts];
  }
  int32_t before = 0, count = 0;  // the expert's pairs in the quarters before this one, and all of them
#pragma unroll
  for (int q = 0; q < kQuarters; ++q) {
    const int32_t v = __shfl(mine, (lane & ~(kQuarters - 1)) + q);
    before += q < quarter ? v : 0;
    count += v;
  }
  // exclusive prefixes over the experts, carried by the first thread of each
  const int32_t pairs = quarter == 0 ? count : 0;
  const int32_t tiles = quarter == 0 ? (count + tile_m - 1) / tile_m : 0;
  int32_t pairs_incl = pairs, tiles_incl = tiles;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int32_t p = __shfl_up(pairs_incl, d), t = __shfl_up(tiles_incl, d);
    if (lane >= d) {
      pairs_incl += p;
      tiles_incl += t;
    }
  }
  if (lane == kWave - 1) {
    s_pairs[wave] = pairs_incl;
    s_tiles[wave] = tiles_incl;
  }
  __syncthreads();
  for (int w = 0; w < wave; ++w) {
    pairs_incl += s_pairs[w];
    tiles_incl += s_tiles[w];
  }
  if (!live) return;
  if (quarter == 0) {
    const int32_t first_tile = tiles_incl - tiles;
    counts[e] = count;
    offsets[e] = pairs_incl - pairs;
    tile_offset[e] = first_tile;
    if (e == n_experts - 1) {
      offsets[n_experts] = pairs_incl;
      tile_offset[n_experts] = min(tiles_incl, max_tiles);
    }
  }
  const int32_t first_tile = __shfl(tiles_incl - tiles, lane & ~(kQuarters - 1));
  const int32_t n_tiles = (count + tile_m - 1) / tile_m;
  for (int t = quarter; t < n_tiles && first_tile + t < max_tiles; t += kQuarters) tile_expert[first_tile + t] = e;
  int b = b_begin;
  for (; b + 8 <= b_end; b += 8) {
    int32_t c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = column[(int64_t)(b + u) * n_experts];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      column[(int64_t)(b + u) * n_experts] = before;
      before += c[u];
    }
  }
  for (; b < b_end; ++b) {
    const int32_t c = column[(int64_t)b * n_experts];
    column[(int64_t)b * n_experts] = before;
    before += c;
  }
}

// The lanes of a wave that hold the same expert id as this one (e < 0: none), from one ballot per bit: ids are below 256.
__device__ __forceinline__ uint64_t lanes_of_expert(int e) {
  uint64_t same = __ballot(e >= 0);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const uint64_t ones = __ballot((e >> bit) & 1);
    same &= ((e >> bit) & 1) ? ones : ~ones;
  }
  return same;
}

__global__ __launch_bounds__(kThreads) void bucket_scatter_kernel(const int32_t* __restrict__ topk_idx,
                                                                  const float* __restrict__ topk_w,
                                                                  int64_t n_pairs, int top_k, int n_experts,
                                                                  const int32_t* __restrict__ block_base,
                                                                  const int32_t* __restrict__ offsets,
                                                                  int32_t* __restrict__ perm,
                                                                  float* __restrict__ w_perm,
                                                                  int32_t* __restrict__ slot_of) {
  // next[w][e]: next free slot of expert e for wave w of this block
  __shared__ int32_t next[kWavesPerBlock][CAMERA_MAX_EXPERTS];
  const int wave = threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  const int64_t block_first = (int64_t)blockIdx.x * kBucketChunk;
  const int64_t wave_first = block_first + (int64_t)wave * kPairsPerWave;

  for (int i = threadIdx.x; i < kWavesPerBlock * CAMERA_MAX_EXPERTS; i += kThreads) (&next[0][0])[i] = 0;
  __syncthreads();
  // per-wave histogram of its own 256 pairs
  for (int it = 0; it < kPairsPerWave / kWave; ++it) {
    const int64_t p = wave_first + it * kWave + lane;
    if (p < n_pairs) {
      const int e = topk_idx[p];
      if (e >= 0 && e < n_experts) atomicAdd(&next[wave][e], 1);
    }
  }
  __syncthreads();
  // turn the histograms into first slots: expert base + block base + earlier waves
  for (int e = threadIdx.x; e < n_experts; e += kThreads) {
    int32_t run = offsets[e] + block_base[(int64_t)blockIdx.x * n_experts + e];
    for (int w = 0; w < kWavesPerBlock; ++w) {
      const int32_t c = next[w][e];
      next[w][e] = run;
      run += c;
    }
  }
  __syncthreads();

  const uint64_t lower_lanes = (1ull << lane) - 1ull;
  for (int it = 0; it < kPairsPerWave / kWave; ++it) {
    const int64_t p = wave_first + it * kWave + lane;
    int e = -1;
    if (p < n_pairs) {
      e = topk_idx[p];
      if (e < 0 || e >= n_experts) e = -1;
    }
    // The lanes that hold the same expert, from one ballot per bit of the id (eight bits: ids are below 256):
    // a lane keeps the lanes that agree with it on every bit.  Its slot is the expert's next free one plus the
    // number of such lanes below it; the lowest lane of every group then moves the expert's counter on.
    const uint64_t same = lanes_of_expert(e);
    int slot = -1;
    if (e >= 0) slot = next[wave][e] + __popcll(same & lower_lanes);
    // every lane has read next[] before the first lane of its group moves it on
    __builtin_amdgcn_wave_barrier();
    if (e >= 0 && (same & lower_lanes) == 0) next[wave][e] += __popcll(same);
    __builtin_amdgcn_wave_barrier();
    if (e >= 0) {
      perm[slot] = (int32_t)(p / top_k);
      if (topk_w) w_perm[slot] = topk_w[p];
    }
    if (slot_of != nullptr && p < n_pairs) slot_of[p] = e >= 0 ? slot : -1;
  }
}

// At most kBucketSmallPairs pairs, one workgroup: a launch and the loads behind it cost more than the counting, which the
// general sort does in three (and a decoding batch needs its work items and appended experts on top).  A wave takes 64
// consecutive pairs, one per lane, and up to four such chunks; the ballots give a pair its place among those of its expert
// in the chunk and the chunk's count; the thread of an expert turns the counts of the chunks into exclusive bases (LDS,
// all loads of a thread in flight); prefixes over the experts follow, pairs and tiles or work items in one pass.
// Replaced, us: the three launches, 1024 pairs of 8 experts 9.6 -> 4.8 (and two gaps), 3176 pairs of 128 experts with the work
// items 19 -> 11; four threads per expert that walked over the pairs, as decoding batches had it, 8 pairs 4.9 -> 4.0, 576
// pairs of 65 experts 14.5 -> 5.0, 1600 of 128 30.7 -> 7.5.  A lone workgroup takes 3 us
// for every thousand pairs and the general sort hardly more for many than for few, so they meet: graph replays of a call that does
// little else, us, three launches / one: 1024 pairs of 8 experts 17.0 / 12.6, 2048 17.2 / 14.3, 3072 17.9 / 17.3, 3584 18.3 / 18.2,
// 4096 18.0 / 18.8, of 128 experts 2048 16.2 / 13.8, 3072 16.2 / 15.9, 3584 16.4 / 17.2, 4096 16.9 / 18.2: the line lies at 3072.
// A decoding batch saves a launch more for its work items and another for appended experts, and stays until 4096: 4096 pairs of 64
// + 2 experts 29.5 / 26.6, of 128 3632 pairs 27.2 / 26.5, 4096 27.3 / 27.8.
// COMPACT: pair token * (top_k + n_shared) + k is routed choice k, or for k >= top_k the appended expert n_experts + k - top_k
// with weight 1; work [2][CAMERA_MAX_EXPERTS + 1] gets the work items.  Otherwise: the M-tile tables.
constexpr int kSmallThreads = 1024;
constexpr int kSmallChunks = kBucketSmallPairs / kWave;
constexpr int kSmallSteps = kBucketSmallPairs / kSmallThreads;
template <bool COMPACT>
__global__ __launch_bounds__(kSmallThreads) void bucket_small_kernel(
    const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w, int n_pairs, int top_k, int n_experts,
    int n_shared, CompactWork tab, int tile_m, int max_tiles, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
    int32_t* __restrict__ tile_offset, int32_t* __restrict__ tile_expert, int32_t* __restrict__ perm,
    float* __restrict__ w_perm, int32_t* __restrict__ slot_of, int32_t* __restrict__ work) {
  __shared__ uint16_t hist[kSmallChunks][CAMERA_MAX_EXPERTS];  // pairs of an expert in a chunk, then in the chunks before it
  __shared__ int32_t first_slot[CAMERA_MAX_EXPERTS];
  constexpr int kExpertWaves = CAMERA_MAX_EXPERTS / kWave;
  __shared__ int32_t wave_total[3][kExpertWaves];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int kk = top_k + n_shared, total = n_experts + n_shared;
  const int n_chunks = (n_pairs + kWave - 1) / kWave;
  for (int i = tid; i < n_chunks * CAMERA_MAX_EXPERTS / 2; i += kSmallThreads) reinterpret_cast<uint32_t*>(&hist[0][0])[i] = 0;
  int expert[kSmallSteps], token[kSmallSteps], place[kSmallSteps];
  float weight[kSmallSteps];
  // pairs past the end have no expert; no early exit, the ballots take whole waves
#pragma unroll
  for (int s = 0; s < kSmallSteps; ++s) {
    const int p = s * kSmallThreads + tid;
    expert[s] = -1;
    weight[s] = 1.0f;
    token[s] = 0;
    if (p < n_pairs) {
      token[s] = p / kk;
      const int k = p - token[s] * kk;
      if (k < top_k) {
        const int e = topk_idx[token[s] * top_k + k];
        if (topk_w) weight[s] = topk_w[token[s] * top_k + k];
        if (e >= 0 && e < n_experts) expert[s] = e;  // an id of the appended experts is not a routed choice
      } else {
        expert[s] = n_experts + k - top_k;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kSmallSteps; ++s) {
    const int chunk = s * (kSmallThreads / kWave) + wave;
    if (chunk >= n_chunks) break;  // wave-uniform
    const uint64_t same = lanes_of_expert(expert[s]);
    place[s] = __popcll(same & ((1ull << lane) - 1ull));
    if (expert[s] >= 0 && place[s] == 0) hist[chunk][expert[s]] = (uint16_t)__popcll(same);
  }
  __syncthreads();
  int32_t value[3] = {0, 0, 0}, incl[3];  // of this thread's expert: pairs; tiles or items of either contraction
  if (tid < total) {
    int run = 0;
    for (int c0 = 0; c0 < n_chunks; c0 += 16) {
      int v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = c0 + u < n_chunks ? hist[c0 + u][tid] : 0;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        if (c0 + u < n_chunks) hist[c0 + u][tid] = (uint16_t)run;
        run += v[u];
      }
    }
    value[0] = run;
    if constexpr (COMPACT) {
      const int groups = (run + kCompactTokens - 1) / kCompactTokens;
      value[1] = groups * tab.hidden_tiles[tid];
      value[2] = groups * tab.down_tiles[tid];
    } else {
      value[1] = (run + tile_m - 1) / tile_m;
    }
  }
  if (wave < kExpertWaves) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      incl[i] = value[i];
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int up = __shfl_up(incl[i], d);
        if (lane >= d) incl[i] += up;
      }
      if (lane == kWave - 1) wave_total[i][wave] = incl[i];
    }
  }
  __syncthreads();
  if (tid < total) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      for (int w = 0; w < wave; ++w) incl[i] += wave_total[i][w];
    first_slot[tid] = incl[0] - value[0];
    counts[tid] = value[0];
    offsets[tid] = incl[0] - value[0];
    if (tid == total - 1) offsets[total] = incl[0];
    if constexpr (COMPACT) {
      int32_t* work2 = work + CAMERA_MAX_EXPERTS + 1;
      work[tid] = incl[1] - value[1];
      work2[tid] = incl[2] - value[2];
      if (tid == total - 1) {
        work[total] = incl[1];
        work2[total] = incl[2];
      }
    } else {
      const int first = incl[1] - value[1];
      tile_offset[tid] = first;
      if (tid == total - 1) tile_offset[total] = min(incl[1], max_tiles);
      for (int t = first; t < min(incl[1], max_tiles); ++t) tile_expert[t] = tid;
    }
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kSmallSteps; ++s) {
    const int p = s * kSmallThreads + tid;
    if (p >= n_pairs) break;
    const int e = expert[s];
    const int slot = e < 0 ? -1 : first_slot[e] + hist[s * (kSmallThreads / kWave) + wave][e] + place[s];
    if (e >= 0) {
      perm[slot] = token[s];
      if (topk_w) w_perm[slot] = weight[s];
    }
    if (slot_of) slot_of[p] = slot;
  }
}

__global__ void dense_tables_kernel(int64_t n, int n_experts, int tile_m, int max_tiles,
                                    int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                    int32_t* __restrict__ tile_offset, int32_t* __restrict__ tile_expert) {
  const int tiles_per = (int)((n + tile_m - 1) / tile_m);
  for (int e = threadIdx.x; e <= n_experts; e += blockDim.x) {
    if (e < n_experts) counts[e] = (int32_t)n;
    offsets[e] = (int32_t)(e * n);
    tile_offset[e] = e * tiles_per;
  }
  for (int t = threadIdx.x; t < n_experts * tiles_per && t < max_tiles; t += blockDim.x)
    tile_expert[t] = t / tiles_per;
}

}  // namespace

hipError_t launch_bucket(hipStream_t stream, const int32_t* topk_idx, const float* topk_w, int64_t n, int top_k,
                         int n_experts, int tile_m, int max_tiles, const BucketTables& t) {
  const int64_t n_pairs = n * top_k;
  if (n_pairs <= kBucketTilesPairs) {
    hipLaunchKernelGGL(bucket_small_kernel<false>, dim3(1), dim3(kSmallThreads), 0, stream, topk_idx, topk_w, (int)n_pairs, top_k,
                       n_experts, 0, CompactWork{}, tile_m, max_tiles, t.counts, t.offsets, t.tile_offset, t.tile_expert, t.perm,
                       t.w_perm, t.slot_of, nullptr);
    return hipGetLastError();
  }
  const int n_blocks = (int)bucket_blocks(n_pairs);
  if (n_blocks > 0)
    hipLaunchKernelGGL(bucket_count_kernel, dim3(n_blocks), dim3(kThreads), 0, stream, topk_idx, n_pairs, n_experts,
                       t.block_hist);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, t.block_hist, n_blocks,
                     n_experts, tile_m, max_tiles, t.counts, t.offsets, t.tile_offset, t.tile_expert);
  if (n_blocks > 0)
    hipLaunchKernelGGL(bucket_scatter_kernel, dim3(n_blocks), dim3(kThreads), 0, stream, topk_idx, topk_w, n_pairs,
                       top_k, n_experts, t.block_hist, t.offsets, t.perm, t.w_perm, t.slot_of);
  return hipGetLastError();
}

hipError_t launch_compact_bucket_small(hipStream_t stream, const int32_t* topk_idx, const float* topk_w, int64_t n,
                                       int top_k, int n_experts, int n_shared, const CompactWork& tab,
                                       const BucketTables& t, int32_t* work) {
  hipLaunchKernelGGL(bucket_small_kernel<true>, dim3(1), dim3(kSmallThreads), 0, stream, topk_idx, topk_w,
                     (int)(n * (top_k + n_shared)), top_k, n_experts, n_shared, tab, 0, 0, t.counts, t.offsets, nullptr, nullptr,
                     t.perm, t.w_perm, t.slot_of, work);
  return hipGetLastError();
}

hipError_t launch_dense_tables(hipStream_t stream, int64_t n, int n_experts, int tile_m, int max_tiles,
                               const BucketTables& t) {
  hipLaunchKernelGGL(dense_tables_kernel, dim3(1), dim3(256), 0, stream, n, n_experts, tile_m, max_tiles, t.counts,
                     t.offsets, t.tile_offset, t.tile_expert);
  return hipGetLastError();
}

}  // namespace camera
