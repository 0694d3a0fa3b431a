// Applying a selection: W_up, W_gate, W_down <- W_up[S,:], W_gate[S,:], W_down[:,S]
// (Algorithm 2, lines 10-13), per expert and packed; with the permutation of
// the bit allocation as the index list it is the reordering that colocates
// micro-experts of equal precision inside an expert (Section "Mixed-precision
// Strategy CAMERA-Q").  Pure data movement, bound by HBM bandwidth:
//   offsets : exclusive prefix of the per-expert entry counts (one small block)
//   rows    : a wave copies one kept gate row and the matching up row, 16 bytes
//             per lane and step -- fully coalesced on both sides
//   columns : a workgroup owns one expert and 16 (or 8) rows of its W_down.  It keeps the expert's column list in
//             LDS and takes R rows at a time through LDS, interleaved: the R values of a column lie side by side, so
//             that one LDS read serves R rows, the loads of R rows are in flight together and there are two barriers
//             per R rows.  A thread takes 16 bytes' worth of output columns and stores 16 bytes in each of the R rows
//             (zeros up to the block's row length, the count rounded up to the caller's row alignment).  The kept
//             columns touch nearly every 64-byte sector of a row, so rows are read whole, with 16-byte loads.
//             Reordering 128 matrices of 2048 x 768 bf16: 211 -> 156 us (5.2 TB/s read and written) against one row
//             at a time with 2-byte LDS reads and stores; keeping 60 % of 64 of 3584 x 2560 and one of 3584 x 20480:
//             571 -> 428 us.  The rows of the two layers: 292 -> 278 and 598 -> 570 us with four vectors of both
//             matrices in flight.
// Entries that do not lie inside their expert give zero rows / columns: no
// address is ever formed from an unchecked index.
#include <hip/hip_bf16.h>

#include "camera_internal.h"

namespace camera {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = kThreads / kWave;  // gather_rows: one wave per output row
constexpr uint16_t kNoColumn = 0xffffu;

// off [n_experts + 1]: prefix of the entry counts; off_ld [n_experts + 1]: prefix of the counts rounded up to
// a multiple of row_align (the row lengths of the W_down blocks).
__global__ __launch_bounds__(CAMERA_MAX_EXPERTS) void gather_offsets_kernel(const int32_t* __restrict__ count,
                                                                            int n_experts, int d_ff, int row_align,
                                                                            int32_t* __restrict__ off,
                                                                            int32_t* __restrict__ off_ld) {
  __shared__ int32_t s_cnt[CAMERA_MAX_EXPERTS];
  const int e = threadIdx.x;
  if (e < n_experts) s_cnt[e] = count ? min(max(count[e], 0), d_ff) : d_ff;
  __syncthreads();
  if (e == 0) {
    int32_t run = 0, run_ld = 0;
    for (int i = 0; i < n_experts; ++i) {
      off[i] = run;
      off_ld[i] = run_ld;
      run += s_cnt[i];
      run_ld += (s_cnt[i] + row_align - 1) / row_align * row_align;
    }
    off[n_experts] = run;
    off_ld[n_experts] = run_ld;
  }
}

// expert that owns output position r: the last e with off[e] <= r (off is non-decreasing, off[0] = 0)
__device__ __forceinline__ int owner_of(const int32_t* s_off, int n_experts, int64_t r) {
  int lo = 0, hi = n_experts;  // invariant: off[lo] <= r < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (s_off[mid] <= r) lo = mid;
    else hi = mid;
  }
  return lo;
}

// row_vecs = d_model * element size / 16.  Output row r of gate_out / up_out <- row index[r] of its expert.
__global__ __launch_bounds__(kThreads) void gather_rows_kernel(
    const u32x4* __restrict__ Wg, const u32x4* __restrict__ Wu, int64_t stride_gu_vecs, int n_experts, int d_ff,
    int row_vecs, const int32_t* __restrict__ index, int64_t n_index, int64_t index_base,
    const int32_t* __restrict__ off, u32x4* __restrict__ gate_out, u32x4* __restrict__ up_out) {
  __shared__ int32_t s_off[CAMERA_MAX_EXPERTS + 1];
  for (int i = threadIdx.x; i <= n_experts; i += kThreads) s_off[i] = off[i];
  __syncthreads();
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int64_t r = (int64_t)blockIdx.x * kRowsPerBlock + wave;
  if (r >= n_index || r >= s_off[n_experts]) return;  // wave-uniform
  const int e = owner_of(s_off, n_experts, r);
  const int64_t c = (int64_t)index[r] - index_base - (int64_t)e * d_ff;
  const bool ok = c >= 0 && c < d_ff;
  const int64_t src = (int64_t)e * stride_gu_vecs + (ok ? c : 0) * row_vecs;
  const int64_t dst = r * row_vecs;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  if (ok && gate_out && up_out) {  // four vectors of both matrices in flight
    for (int k0 = lane; k0 < row_vecs; k0 += 4 * kWave) {
      u32x4 g[4], u[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k0 + i * kWave >= row_vecs) continue;
        g[i] = __builtin_nontemporal_load(&Wg[src + k0 + i * kWave]);
        u[i] = __builtin_nontemporal_load(&Wu[src + k0 + i * kWave]);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (k0 + i * kWave >= row_vecs) continue;
        __builtin_nontemporal_store(g[i], &gate_out[dst + k0 + i * kWave]);
        __builtin_nontemporal_store(u[i], &up_out[dst + k0 + i * kWave]);
      }
    }
    return;
  }
  for (int k = lane; k < row_vecs; k += kWave) {
    if (gate_out) gate_out[dst + k] = ok ? Wg[src + k] : zero;
    if (up_out) up_out[dst + k] = ok ? Wu[src + k] : zero;
  }
}

// T: element type by size (uint16_t for bf16, uint32_t for float32).  R: rows taken through LDS at a time.  VEC: rows of
// W_down start on 16-byte boundaries and are whole 16-byte vectors long.  store_vec: down_out is 16-byte aligned.
// Dynamic LDS: d_ff columns of R elements of T, then the column list, uint16, filled up to whole groups of V columns.
template <class T, int R>
struct alignas(sizeof(T) * R) RowSet {
  T v[R];
};
template <class T, int R, bool VEC>
__global__ void gather_cols_kernel(const T* __restrict__ Wd, int64_t stride_down, int d_ff, int d_model,
                                   const int32_t* __restrict__ index, int64_t n_index, int64_t index_base,
                                   const int32_t* __restrict__ off, const int32_t* __restrict__ off_ld,
                                   int rows_per_block, bool store_vec, T* __restrict__ down_out) {
  constexpr int V = 16 / sizeof(T);  // elements of a 16-byte vector
  using Vec = __attribute__((ext_vector_type(V))) T;
  using Cols = __attribute__((ext_vector_type(V))) uint16_t;
  extern __shared__ __align__(16) unsigned char smem[];
  RowSet<T, R>* s_set = reinterpret_cast<RowSet<T, R>*>(smem);
  uint16_t* s_col = reinterpret_cast<uint16_t*>(smem + (((size_t)d_ff * sizeof(T) * R + 15) & ~size_t(15)));
  const int tid = threadIdx.x, n_threads = blockDim.x;
  const int e = blockIdx.x;
  const int64_t first = off[e];
  const int cnt = (int)min((int64_t)(off[e + 1] - off[e]), max((int64_t)0, n_index - first));  // entries that exist
  if (cnt <= 0) return;  // block-uniform
  for (int j = tid; j < (cnt + V - 1) / V * V; j += n_threads) {
    const int64_t c = j < cnt ? (int64_t)index[first + j] - index_base - (int64_t)e * d_ff : -1;
    s_col[j] = (c >= 0 && c < d_ff) ? (uint16_t)c : kNoColumn;  // d_ff <= 32768 (checked by the caller), so no clash
  }
  const T* src_expert = Wd + (int64_t)e * stride_down;
  const int ld = off_ld[e + 1] - off_ld[e];  // row length of the block: the count rounded up, the rest zero
  T* dst_expert = down_out + off_ld[e] * (int64_t)d_model;
  const int r_begin = blockIdx.y * rows_per_block, r_end = min(d_model, r_begin + rows_per_block);
  for (int r = r_begin; r < r_end; r += R) {
    __syncthreads();  // the column list is complete; the previous rows have been read out
    const T* src_row[R];
#pragma unroll
    for (int i = 0; i < R; ++i) src_row[i] = src_expert + (int64_t)min(r + i, r_end - 1) * d_ff;
    if (VEC) {
      for (int k = tid; k < d_ff / V; k += n_threads) {
        Vec in[R];
#pragma unroll
        for (int i = 0; i < R; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(src_row[i]) + k);
#pragma unroll
        for (int c = 0; c < V; ++c) {
          RowSet<T, R> set;
#pragma unroll
          for (int i = 0; i < R; ++i) set.v[i] = in[i][c];
          s_set[k * V + c] = set;
        }
      }
    } else {
      for (int k = tid; k < d_ff; k += n_threads) {
        RowSet<T, R> set;
#pragma unroll
        for (int i = 0; i < R; ++i) set.v[i] = src_row[i][k];
        s_set[k] = set;
      }
    }
    __syncthreads();
    T* dst_row = dst_expert + (int64_t)r * ld;
    const int rows = min(R, r_end - r);
    if (store_vec && ld % V == 0) {  // block-uniform; off_ld * d_model is whole vectors, so every row starts on one
      for (int j = tid; j < ld / V; j += n_threads) {
        Vec out[R];
        Cols col;
        if (j * V < cnt) {
          col = *reinterpret_cast<const Cols*>(s_col + j * V);
        } else {
#pragma unroll
          for (int c = 0; c < V; ++c) col[c] = kNoColumn;
        }
#pragma unroll
        for (int c = 0; c < V; ++c) {
          const bool have = col[c] != kNoColumn;
          const RowSet<T, R> set = s_set[have ? col[c] : 0];
#pragma unroll
          for (int i = 0; i < R; ++i) out[i][c] = have ? set.v[i] : T(0);
        }
#pragma unroll
        for (int i = 0; i < R; ++i)
          if (i < rows) __builtin_nontemporal_store(out[i], reinterpret_cast<Vec*>(dst_row + (int64_t)i * ld) + j);
      }
    } else {
      for (int j = tid; j < ld; j += n_threads) {
        const uint16_t c = j < cnt ? s_col[j] : kNoColumn;
        const bool have = c != kNoColumn;
        const RowSet<T, R> set = s_set[have ? c : 0];
#pragma unroll
        for (int i = 0; i < R; ++i)
          if (i < rows) dst_row[(int64_t)i * ld + j] = have ? set.v[i] : T(0);
      }
    }
  }
}

}  // namespace

hipError_t launch_gather_offsets(hipStream_t stream, const int32_t* count, int n_experts, int64_t d_ff,
                                 int row_align, int32_t* off, int32_t* off_ld) {
  hipLaunchKernelGGL(gather_offsets_kernel, dim3(1), dim3(CAMERA_MAX_EXPERTS), 0, stream, count, n_experts, (int)d_ff,
                     row_align, off, off_ld);
  return hipGetLastError();
}

hipError_t launch_gather_rows(hipStream_t stream, int dtype, const void* W_gate, const void* W_up, int64_t stride_gu,
                              int n_experts, int64_t d_ff, int64_t d_model, const int32_t* index, int64_t n_index,
                              int64_t index_base, const int32_t* off, void* gate_out, void* up_out) {
  if (n_index <= 0 || (gate_out == nullptr && up_out == nullptr)) return hipSuccess;
  const int es = dtype == CAMERA_BF16 ? 2 : 4;
  const int64_t blocks = (n_index + kRowsPerBlock - 1) / kRowsPerBlock;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream,
                     static_cast<const u32x4*>(W_gate), static_cast<const u32x4*>(W_up), stride_gu * es / 16, n_experts,
                     (int)d_ff, (int)(d_model * es / 16), index, n_index, index_base, off,
                     static_cast<u32x4*>(gate_out), static_cast<u32x4*>(up_out));
  return hipGetLastError();
}

template <class T, int R>
static hipError_t launch_cols_of(hipStream_t stream, const void* W_down, int64_t stride_down, int n_experts,
                                 int64_t d_ff, int64_t d_model, const int32_t* index, int64_t n_index,
                                 int64_t index_base, const int32_t* off, const int32_t* off_ld, size_t smem,
                                 void* down_out) {
  const bool vec = (d_ff * sizeof(T)) % 16 == 0 && (stride_down * sizeof(T)) % 16 == 0 &&
                   (reinterpret_cast<uintptr_t>(W_down) & 15u) == 0;
  auto kern = vec ? gather_cols_kernel<T, R, true> : gather_cols_kernel<T, R, false>;
  hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
  if (err != hipSuccess) return err;
  // 16 rows share a column list; 8 where 16 would leave the chip short of workgroups (one wide shared expert)
  const int rows = n_experts * d_model >= 16 * 2048 ? 16 : 8;
  // few workgroups fit a CU: larger ones fill it; a row of one wave's elements leaves the other waves idle
  const int threads = d_ff <= kWave ? kWave : (smem <= 40 * 1024 ? kThreads : 4 * kThreads);
  dim3 grid((unsigned)n_experts, (unsigned)((d_model + rows - 1) / rows));
  hipLaunchKernelGGL(kern, grid, dim3(threads), smem, stream, static_cast<const T*>(W_down), stride_down, (int)d_ff,
                     (int)d_model, index, n_index, index_base, off, off_ld, rows,
                     (reinterpret_cast<uintptr_t>(down_out) & 15u) == 0, static_cast<T*>(down_out));
  return hipGetLastError();
}

template <class T>
static hipError_t launch_cols(hipStream_t stream, const void* W_down, int64_t stride_down, int n_experts, int64_t d_ff,
                              int64_t d_model, const int32_t* index, int64_t n_index, int64_t index_base,
                              const int32_t* off, const int32_t* off_ld, void* down_out) {
  // rows through LDS at a time: the more, the fewer LDS accesses and barriers, as long as two workgroups fit a CU's
  // 160 KiB; a row of at most 64 KiB and its column list (at most 32768 entries) always fit alone
  auto smem = [&](int r) {
    return (((size_t)d_ff * sizeof(T) * r + 15) & ~size_t(15)) + (((size_t)d_ff + 7) & ~size_t(7)) * sizeof(uint16_t);
  };
  constexpr size_t kTwoPerCu = 80 * 1024;
  if (smem(4) <= kTwoPerCu)
    return launch_cols_of<T, 4>(stream, W_down, stride_down, n_experts, d_ff, d_model, index, n_index, index_base, off,
                                off_ld, smem(4), down_out);
  if (smem(2) <= kTwoPerCu)
    return launch_cols_of<T, 2>(stream, W_down, stride_down, n_experts, d_ff, d_model, index, n_index, index_base, off,
                                off_ld, smem(2), down_out);
  return launch_cols_of<T, 1>(stream, W_down, stride_down, n_experts, d_ff, d_model, index, n_index, index_base, off,
                              off_ld, smem(1), down_out);
}

hipError_t launch_gather_cols(hipStream_t stream, int dtype, const void* W_down, int64_t stride_down, int n_experts,
                              int64_t d_ff, int64_t d_model, const int32_t* index, int64_t n_index,
                              int64_t index_base, const int32_t* off, const int32_t* off_ld, void* down_out) {
  if (n_index <= 0 || down_out == nullptr) return hipSuccess;
  if (dtype == CAMERA_BF16)
    return launch_cols<uint16_t>(stream, W_down, stride_down, n_experts, d_ff, d_model, index, n_index, index_base, off,
                                 off_ld, down_out);
  return launch_cols<uint32_t>(stream, W_down, stride_down, n_experts, d_ff, d_model, index, n_index, index_base, off,
                               off_ld, down_out);
}

}  // namespace camera
