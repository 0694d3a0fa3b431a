// The layer output from compacted weights (the result of Algorithm 2, lines
// 10-13: every expert keeps its own number of micro-experts), for the small
// token batches of decoding (the setting of the decoding-speed comparison of a
// pruned MoE layer, batch of 64 tokens).
//
// With a handful of tokens per expert the layer is bound by reading each
// activated expert's weights once, so no operand is tiled through LDS: a
// workgroup owns 32 weight rows and up to 32 tokens of one expert, its waves
// split the K extent between them and stream their share from HBM straight
// into MFMA operand registers (the weight rows are the M side, the tokens the
// N side); the partial sums of the waves meet in
// LDS, added in wave order.  Work items are kept small and alike, so that a
// launch has several times more workgroups than the chip holds at once and its
// last round does not leave most compute units idle:
//   - the K extent of a workgroup is split between its waves;
//   - the 32-token groups of an expert go to different workgroups, eight apart
//     in the launch: on the same XCD and at about the same time, so that its L2
//     serves the weights to all but the first of them;
//   - in the second contraction an expert with many kept micro-experts (a
//     large shared expert) is cut into K chunks that go to different
//     workgroups, each writing its own partial product rows; the chunks are
//     added, in chunk order, when the token's experts are summed.
// Operands are those of v_mfma_f32_16x16x32_bf16, two weight-row tiles by one or
// two token tiles per wave: lane (row, quarter) loads 16 bytes and the four
// lanes of a row read one whole 64-byte sector, so that a sector is asked for
// by one instruction only.  (With 32x32x16 operands two lanes share a row: 64
// tokens of the Qwen2 shape, 40 % pruned, took 341 + 220 us, now 314 + 194 us.
// Of that layer unpruned the vector caches ask their L2 for 28.0 and 16.4 million
// reads where the kernels before this form and its work items asked for 29.2 and
// 17.0, and memory is read 1.02 and 1.05 times the weights, before 1.13 and 1.15.
// Those few per cent are what the counters show; the rest of the gain was not
// traced to a cause.)  A group of at
// most 16 tokens leaves out the second token tile.  Experts that no token of
// the batch selected are skipped before any weight is read.
//
//   hidden  : Lambda[slot][c] = a silu(x w_gate,c) (x w_up,c), bf16, for the c < count[e] kept micro-experts
//   down    : partial[chunk][slot][r] = sum over the chunk's c of Lambda[slot][c] W_down_e[r][c], float32
//   combine : y_token (+)= the partial rows of its experts' slots, experts in k order, chunks in chunk order
// The rows of the compacted W_down block of an expert hold count[e] elements and
// then zeros up to the caller's row alignment.  Without alignment (rows of any
// length) its 16-byte loads are unaligned (2-byte aligned) and the chunk that
// straddles the end of a row is taken as the 16 bytes that end there, shifted
// down: correct, but a third slower than rows that start on 128-byte lines.
#include "camera_internal.h"

namespace camera {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;

// Waves of a workgroup, each with its share of the K blocks (1, 2 or 4: the four accumulator groups of a lane
// are dealt to them after the reduction).  The first contraction's K extent is d_model.
#ifndef CAMERA_COMPACT_KSPLIT_HIDDEN
#define CAMERA_COMPACT_KSPLIT_HIDDEN 4
#endif
constexpr int kSplitHidden = CAMERA_COMPACT_KSPLIT_HIDDEN;
static_assert(kSplitHidden == 1 || kSplitHidden == 2 || kSplitHidden == 4, "1, 2 or 4 waves");
// The second contraction's K extent is the expert's kept count, which shrinks with the pruning ratio: four
// waves while a K chunk gives each of them at least five K blocks, two below that (measured 3-8 % apart).
constexpr int kDownFourWavesFrom = 1280;
constexpr int kTile = 16;    // rows and columns of an MFMA
constexpr int kRows = 32;    // weight rows per workgroup: two M tiles
constexpr int kTokens = kCompactTokens;  // tokens per workgroup: one or two N tiles
constexpr int kKBlock = 64;  // K elements per step: 2 MFMAs of K = 32 per pair of tiles

__device__ __forceinline__ float silu_f32(float g) {
  return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f));
}

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
  return z;
}

// 16 bytes from a 16-byte aligned address
__device__ __forceinline__ bf16x8 load8(const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }
// 16 bytes from an address that is only element aligned
__device__ __forceinline__ bf16x8 load8_unaligned(const __bf16* p) {
  bf16x8 v;
  __builtin_memcpy(&v, p, sizeof(v));
  return v;
}

// One lane's share of a 64-element K block of two 16-row tiles: c[i][s] covers elements [32 s + 8 q, 32 s + 8 q + 8) of
// row 16 i + r, for lane = 16 q + r.
struct Frag {
  bf16x8 c[2][2];
};
// p: the row's first element of the block (for s = 0) of this lane's quarter
template <bool ALIGNED>
__device__ __forceinline__ void load_rows(bf16x8 (&c)[2], const __bf16* p) {
#pragma unroll
  for (int s = 0; s < 2; ++s) c[s] = ALIGNED ? load8(p + 32 * s) : load8_unaligned(p + 32 * s);
}

// out[i] = w[i + d] for i + d < 8, else 0 (1 <= d <= 7, the same for the whole wave)
__device__ __forceinline__ bf16x8 shift_down(bf16x8 w, int d) {
  const u64x2 v = __builtin_bit_cast(u64x2, w);
  const int s = 16 * d;
  u64x2 o;
  if (s < 64) {
    o[0] = (v[0] >> s) | (v[1] << (64 - s));
    o[1] = v[1] >> s;
  } else {
    o[0] = v[1] >> (s - 64);
    o[1] = 0;
  }
  return __builtin_bit_cast(bf16x8, o);
}

// The last, partial K block of an operand row.  `k` is the K index (inside the block) of the lane's first element,
// `k_full` the end of the valid elements.  MODE says what lies behind k_full:
//   kWhole   k_full is a multiple of 8 (no partial chunk)
//   kPadded  the row is zero-filled and readable up to the next multiple of 8
//   kRagged  nothing at or beyond k_full may be touched: the chunk that straddles the end is taken as the 16 bytes
//            that end at k_full, shifted down (`row_k`, the valid elements of the whole row, must be >= 8 for
//            that; shorter rows are read element by element)
enum TailMode { kWhole, kPadded, kRagged };
template <bool ALIGNED, TailMode MODE>
__device__ __forceinline__ void load_rows_tail(bf16x8 (&c)[2], const __bf16* p, int k, int k_full, int row_k) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int kj = k + 32 * j;
    const __bf16* pj = p + 32 * j;
    if (kj + 8 <= k_full || (MODE == kPadded && kj < k_full)) {
      c[j] = ALIGNED ? load8(pj) : load8_unaligned(pj);
    } else if (MODE == kRagged && kj < k_full) {
      const int valid = k_full - kj;  // 1..7, the same for every lane that gets here
      if (row_k >= 8) {
        c[j] = shift_down(load8_unaligned(pj + valid - 8), 8 - valid);
      } else {
        u64x2 o = {0, 0};
#pragma unroll 1
        for (int i = 0; i < valid; ++i) {
          const uint64_t x = __builtin_bit_cast(uint16_t, pj[i]);
          o[i >> 2] |= x << (16 * (i & 3));
        }
        c[j] = __builtin_bit_cast(bf16x8, o);
      }
    } else {
      c[j] = zero8();
    }
  }
}

// acc.t[i][n]: weight tile i by token tile n.  Element e of a lane: weight row 16 i + 4 (lane / 16) + e, token 16 n + lane % 16.
struct Acc {
  f32x4 t[2][2] = {};
};
template <int NT>
__device__ __forceinline__ void multiply(Acc& acc, const Frag& a, const Frag& b) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int n = 0; n < NT; ++n)
        acc.t[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.c[i][s], b.c[n][s], acc.t[i][n], 0, 0, 0);
}

// ---- partial sums of the waves ------------------------------------------------------------------------------
// red[wave][m][4 g + e][lane]: element e of `lane` in group g = 2 i + n of product m.  With one wave per workgroup nothing goes through LDS.
template <int KS, int TILES>
struct Reduce {
  float (*red)[TILES][16][kWave];
  __device__ __forceinline__ void put(int wave, int tile, const Acc& acc, int lane) const {
#pragma unroll
    for (int i = 0; i < 16; ++i) red[wave][tile][i][lane] = acc.t[i / 8][i / 4 % 2][i % 4];
  }
  __device__ __forceinline__ float get(int tile, int i, int lane) const {
    float s = red[0][tile][i][lane];
#pragma unroll
    for (int w = 1; w < KS; ++w) s += red[w][tile][i][lane];
    return s;
  }
};
// The groups of four accumulator elements that `wave` finishes after the reduction.
template <int KS>
__device__ __forceinline__ bool owns_group(int wave, int q) { return (q * KS) / 4 == wave; }

// K blocks [kb0, kb1) of a wave; the wave with `tail` also takes the partial block after the last full one.
struct KRange {
  int kb0, kb1;
  bool tail;
};
template <int KS>
__device__ __forceinline__ KRange k_range(int full_blocks, bool has_tail, int wave) {
  KRange k;
  k.kb0 = full_blocks * wave / KS;
  k.kb1 = full_blocks * (wave + 1) / KS;
  k.tail = has_tail && wave == KS - 1;
  return k;
}

// ---- work items -----------------------------------------------------------------------------------------------
// A work item is one weight tile of one expert with one group of kTokens of the expert's tokens.  work_off[e], the items
// of the experts before e (work_off[n_experts]: all items), is made on the device with the bucket order, because only
// there the groups of an expert are known; the host launches an upper bound.  (A grid of tiles x token groups of the
// batch is mostly workgroups of groups that an expert does not have: 23 of 24 at 397 tokens and 128 experts, and
// starting them cost more than a fifth of the two kernels.)
struct WorkItem {
  int e, tile, group;  // tile inside the expert
};
// All lanes of a wave call it with the same id < work_off[n_experts]: lane l looks at experts l, l + 64, ...
__device__ __forceinline__ int find_expert(const int32_t* __restrict__ work_off, int n_experts, int id) {
  const int lane = threadIdx.x & 63;
  int e = 0;
#pragma unroll
  for (int i = 0; i < CAMERA_MAX_EXPERTS / kWave; ++i) {
    const int at = i * kWave + lane + 1;
    e += __popcll(__ballot(at < n_experts && work_off[min(at, n_experts)] <= id));
  }
  return __builtin_amdgcn_readfirstlane(e);
}
// Eight tiles, then the next group of the same eight: workgroup ids go round the eight XCDs, so the groups of a tile
// stay on one.
__device__ __forceinline__ WorkItem item_of(int e, int local, int tiles, int groups) {
  constexpr int kXcds = 8;
  WorkItem w;
  w.e = e;
  const int block = local / (kXcds * groups);
  const int width = min(kXcds, tiles - block * kXcds);  // the last tiles of an expert may be fewer than eight
  const int in = local - block * kXcds * groups;
  w.group = in / width;
  w.tile = block * kXcds + in - w.group * width;
  return w;
}
__device__ __forceinline__ int groups_of(int m) { return (m + kTokens - 1) / kTokens; }

// Exclusive prefix over the threads of a workgroup of WAVES waves.  s_total: one entry per wave.
template <int WAVES>
__device__ __forceinline__ int block_prefix(int mine, int32_t* s_total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = mine;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  __syncthreads();  // s_total may hold an earlier call's totals
  if (lane == kWave - 1) s_total[wave] = incl;
  __syncthreads();
  int first = incl - mine;
  for (int w = 0; w < wave; ++w) first += s_total[w];
  return first;
}
// work [2][CAMERA_MAX_EXPERTS + 1]: the items of the first contraction (32-row tiles of the kept rows), then of the
// second (K chunks x 32-row tiles of d_model).  Thread e < total has expert e with m tokens.
template <int WAVES>
__device__ __forceinline__ void write_work(const CompactWork& tab, int total, int m, int32_t* s_total,
                                           int32_t* __restrict__ work) {
  const int e = threadIdx.x;
  const int g = e < total ? groups_of(m) : 0;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    const int mine = e < total ? g * (which ? tab.down_tiles[e] : tab.hidden_tiles[e]) : 0;
    const int first = block_prefix<WAVES>(mine, s_total);
    int32_t* out = work + which * (CAMERA_MAX_EXPERTS + 1);
    if (e < total) out[e] = first;
    if (e == total - 1) out[total] = first + mine;
  }
}

// ---- Lambda = a silu(X W_gate^T) (X W_up^T) on the kept rows ----------------------------------------------
// wg, wu, x: the two rows of a lane (of tiles 0 and 1), at the lane's quarter of the first K block
template <int NT>
__device__ __forceinline__ void hidden_pass(const __bf16* const (&wg)[2], const __bf16* const (&wu)[2],
                                            const __bf16* const (&x)[2], int d_model, KRange kr, Acc& g, Acc& u) {
  Frag ag[2], au[2], b[2];
  auto fetch = [&](int buf, int kb) {
    const int off = kb * kKBlock;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      load_rows<true>(ag[buf].c[i], wg[i] + off);
      load_rows<true>(au[buf].c[i], wu[i] + off);
      if (i < NT) load_rows<true>(b[buf].c[i], x[i] + off);
    }
  };
  auto both = [&](int buf) {
    multiply<NT>(g, ag[buf], b[buf]);
    multiply<NT>(u, au[buf], b[buf]);
  };
  int kb = kr.kb0;
  if (kb < kr.kb1) fetch(0, kb);
  for (; kb + 2 <= kr.kb1; kb += 2) {  // the loads of the next block are in flight while this one multiplies
    fetch(1, kb + 1);
    both(0);
    if (kb + 2 < kr.kb1) fetch(0, kb + 2);
    both(1);
  }
  if (kb < kr.kb1) both(0);
  if (kr.tail) {
    const int full = d_model / kKBlock;
    const int rem = d_model - full * kKBlock;     // a multiple of 8
    const int k = (threadIdx.x & 63) / kTile * 8;  // K index of the lane's first element inside the block
    const int off = full * kKBlock;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      load_rows_tail<true, kWhole>(ag[0].c[i], wg[i] + off, k, rem, d_model);
      load_rows_tail<true, kWhole>(au[0].c[i], wu[i] + off, k, rem, d_model);
      if (i < NT) load_rows_tail<true, kWhole>(b[0].c[i], x[i] + off, k, rem, d_model);
    }
    both(0);
  }
}

// Workgroups take the items blockIdx.x, blockIdx.x + gridDim.x, ...
template <int KS>
__global__ __launch_bounds__(kWave * KS) __attribute__((amdgpu_waves_per_eu(2))) void compact_hidden_kernel(
    const __bf16* __restrict__ X, int64_t ldx, int d_model, const __bf16* __restrict__ W_gate,
    const __bf16* __restrict__ W_up, CompactRows tab, const int32_t* __restrict__ work_off,
    const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets, const int32_t* __restrict__ perm,
    const float* __restrict__ w_perm, __bf16* __restrict__ H, int ldh) {
  __shared__ float red_mem[KS][2][16][kWave];  // gate and up
  const Reduce<KS, 2> red{red_mem};
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r = lane % kTile, q = lane / kTile;
  const KRange kr = k_range<KS>(d_model / kKBlock, d_model % kKBlock != 0, wave);
  const int n_items = work_off[tab.n_experts];
  for (int id = blockIdx.x; id < n_items; id += gridDim.x) {
    const int e = find_expert(work_off, tab.n_experts, id);
    const int m = __builtin_amdgcn_readfirstlane(counts[e]);
    const int slot0 = __builtin_amdgcn_readfirstlane(offsets[e]);
    const WorkItem w = item_of(e, id - work_off[e], tab.tile_off[e + 1] - tab.tile_off[e], groups_of(m));
    const int cnt = tab.row_off[e + 1] - tab.row_off[e];
    const int cnt8 = (cnt + 7) & ~7;
    const int c0 = w.tile * kRows;
    const int t0 = w.group * kTokens;
    const __bf16 *wg[2], *wu[2], *x[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = min(c0 + kTile * i + r, cnt - 1);  // rows past the expert's end repeat its last row, columns past m
      const int tc = min(t0 + kTile * i + r, m - 1);     // its last token; their results are dropped
      const int64_t w_at = ((int64_t)tab.row_off[e] + row) * d_model + q * 8;
      wg[i] = W_gate + w_at;
      wu[i] = W_up + w_at;
      x[i] = X + (int64_t)(perm ? perm[slot0 + tc] : tc) * ldx + q * 8;
    }
    Acc g, u;
    if (m - t0 > kTile)
      hidden_pass<2>(wg, wu, x, d_model, kr, g, u);
    else
      hidden_pass<1>(wg, wu, x, d_model, kr, g, u);
    if constexpr (KS > 1) {
      red.put(wave, 0, g, lane);
      red.put(wave, 1, u, lane);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int group = 2 * i + n;
        const int t = t0 + kTile * n + r;
        const int c = c0 + kTile * i + 4 * q;
        // columns [cnt, cnt8) are written as zeros: the down kernel reads whole chunks
        if (!owns_group<KS>(wave, group) || t >= m || c >= cnt8) continue;
        const int64_t slot = slot0 + t;
        const float a = w_perm ? w_perm[slot] : 1.0f;
        bf16x4 out;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float gv = KS > 1 ? red.get(0, 4 * group + k, lane) : g.t[i][n][k];
          const float uv = KS > 1 ? red.get(1, 4 * group + k, lane) : u.t[i][n][k];
          const float lam = a * silu_f32(gv) * uv;
          out[k] = (__bf16)(c + k < cnt ? lam : 0.0f);
        }
        *reinterpret_cast<bf16x4*>(H + slot * ldh + c) = out;
      }
    }
    if constexpr (KS > 1) __syncthreads();  // the next item writes the same LDS
  }
}

// ---- partial = Lambda W_down_e^T over one K chunk ----------------------------------------------------------
// wd, hrow: the two rows of a lane, at the lane's quarter of the chunk's first K block; k_len: the chunk's length; row_k:
// the valid length of the whole row.
template <int NT>
__device__ __forceinline__ void down_pass(const __bf16* const (&wd)[2], const __bf16* const (&hrow)[2], int k_len,
                                          int row_k, KRange kr, Acc& p) {
  Frag a[2], b[2];
  auto fetch = [&](int buf, int kb) {
    const int off = kb * kKBlock;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      load_rows<false>(a[buf].c[i], wd[i] + off);
      if (i < NT) load_rows<true>(b[buf].c[i], hrow[i] + off);
    }
  };
  int kb = kr.kb0;
  if (kb < kr.kb1) fetch(0, kb);
  for (; kb + 2 <= kr.kb1; kb += 2) {
    fetch(1, kb + 1);
    multiply<NT>(p, a[0], b[0]);
    if (kb + 2 < kr.kb1) fetch(0, kb + 2);
    multiply<NT>(p, a[1], b[1]);
  }
  if (kb < kr.kb1) multiply<NT>(p, a[0], b[0]);
  if (kr.tail) {
    const int full = k_len / kKBlock;
    const int rem = k_len - full * kKBlock;
    const int k = (threadIdx.x & 63) / kTile * 8;
    const int off = full * kKBlock;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      load_rows_tail<false, kRagged>(a[0].c[i], wd[i] + off, k, rem, row_k);  // never past the end of the weight row
      // Lambda rows are zero-filled up to a multiple of 8
      if (i < NT) load_rows_tail<true, kPadded>(b[0].c[i], hrow[i] + off, k, rem, row_k);
    }
    multiply<NT>(p, a[0], b[0]);
  }
}

// Length of the K chunks of an expert with cnt kept micro-experts cut into n_chunks (a multiple of 64).
__device__ __forceinline__ int chunk_length(int cnt, int n_chunks) {
  return ((cnt + n_chunks - 1) / n_chunks + kKBlock - 1) & ~(kKBlock - 1);
}

// The tiles of an expert are (K chunk, 32-row tile of d_model).  partial is [chunk within the expert][n_slots][d_model].
template <int KS>
__global__ __launch_bounds__(kWave * KS) __attribute__((amdgpu_waves_per_eu(3))) void compact_down_kernel(
    const __bf16* __restrict__ H, int ldh, const __bf16* __restrict__ W_down, int d_model, CompactDown tab,
    const int32_t* __restrict__ work_off, const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets, int64_t n_slots,
    float* __restrict__ partial) {
  __shared__ float red_mem[KS][1][16][kWave];
  const Reduce<KS, 1> red{red_mem};
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int row_tiles = (d_model + kRows - 1) / kRows;
  const int r = lane % kTile, q = lane / kTile;
  const int n_items = work_off[tab.n_experts];
  for (int id = blockIdx.x; id < n_items; id += gridDim.x) {
    const int e = find_expert(work_off, tab.n_experts, id);
    const int m = __builtin_amdgcn_readfirstlane(counts[e]);
    const int slot0 = __builtin_amdgcn_readfirstlane(offsets[e]);
    const int n_chunks = tab.chunk_off[e + 1] - tab.chunk_off[e];
    const WorkItem w = item_of(e, id - work_off[e], n_chunks * row_tiles, groups_of(m));
    const int cnt = tab.count[e];
    const int ld = tab.ld_off[e + 1] - tab.ld_off[e];  // row length of the expert's block (cnt and zero padding)
    const int chunk_in = w.tile / row_tiles;
    const int r0 = (w.tile - chunk_in * row_tiles) * kRows;
    const int len = chunk_length(cnt, n_chunks);
    const int k0 = min(chunk_in * len, cnt);
    const int k_len = min(len, cnt - k0);
    const KRange kr = k_range<KS>(k_len / kKBlock, k_len % kKBlock != 0, wave);
    float* out_chunk = partial + (int64_t)chunk_in * n_slots * d_model;
    const int t0 = w.group * kTokens;
    const __bf16 *wd[2], *hrow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = min(r0 + kTile * i + r, d_model - 1);
      wd[i] = W_down + (int64_t)tab.ld_off[e] * d_model + (int64_t)row * ld + k0 + q * 8;
      hrow[i] = H + (int64_t)(slot0 + min(t0 + kTile * i + r, m - 1)) * ldh + k0 + q * 8;
    }
    Acc p;
    if (m - t0 > kTile)
      down_pass<2>(wd, hrow, k_len, cnt, kr, p);
    else
      down_pass<1>(wd, hrow, k_len, cnt, kr, p);
    if constexpr (KS > 1) {
      red.put(wave, 0, p, lane);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int group = 2 * i + n;
        const int t = t0 + kTile * n + r;
        const int rr = r0 + kTile * i + 4 * q;
        // d_model is a multiple of 8: four rows are inside or outside as a whole
        if (!owns_group<KS>(wave, group) || t >= m || rr >= d_model) continue;
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = KS > 1 ? red.get(0, 4 * group + k, lane) : p.t[i][n][k];
        *reinterpret_cast<float4*>(out_chunk + (int64_t)(slot0 + t) * d_model + rr) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
    if constexpr (KS > 1) __syncthreads();  // the next item writes the same LDS
  }
}

// ---- y_token (+)= its partial rows -------------------------------------------------------------------------
// grid: x = tokens, y = blockDim.x vectors of four columns each.  Routed: the token's slots are
// slot_of[token * terms + k], of expert topk_idx[token][k] for k < top_k and n_routed + k - top_k beyond; dense
// (slot_of == nullptr): expert k, slot k * n + token.  A workgroup has one token, so slots, experts and chunk counts are
// scalar loads; the first chunks of eight terms are in flight together, then the further chunks of a term.  (One thread
// per output that searched the expert of every slot in turn was a chain of some sixty dependent loads:
// 1 token 12 -> 6 us, 64 tokens of the Qwen2 shape 21 -> 10 us, 397 of the Qwen3 shape 22 -> 8 us.)
constexpr int kTerms = 8;
__device__ __forceinline__ void add4(float4& s, const float4& p) {
  s.x += p.x;
  s.y += p.y;
  s.z += p.z;
  s.w += p.w;
}
__global__ __launch_bounds__(256) void compact_combine_kernel(const float4* __restrict__ partial,
                                                              const int32_t* __restrict__ slot_of,
                                                              const int32_t* __restrict__ topk_idx, CompactDown tab,
                                                              int64_t n, int terms, int top_k, int n_routed, int vecs,
                                                              int64_t n_slots, int accumulate, float4* __restrict__ Y) {
  const int64_t tok = blockIdx.x;
  const int v = (int)(blockIdx.y * blockDim.x + threadIdx.x);
  if (v >= vecs) return;
  float4 s = accumulate ? Y[tok * vecs + v] : make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < terms; k0 += kTerms) {
    int64_t slot[kTerms];
    int chunks[kTerms];
    float4 p[kTerms];
#pragma unroll
    for (int u = 0; u < kTerms; ++u) {
      const int k = k0 + u;
      chunks[u] = 0;
      slot[u] = -1;
      if (k >= terms) continue;
      int e = k;
      if (slot_of) {
        slot[u] = slot_of[tok * terms + k];
        e = k < top_k ? topk_idx[tok * top_k + k] : n_routed + k - top_k;
      } else {
        slot[u] = (int64_t)k * n + tok;
      }
      if (slot[u] >= 0) chunks[u] = tab.chunk_off[e + 1] - tab.chunk_off[e];  // below 0: an expert id outside the group
    }
#pragma unroll
    for (int u = 0; u < kTerms; ++u)
      if (chunks[u] > 0) p[u] = partial[slot[u] * vecs + v];
#pragma unroll
    for (int u = 0; u < kTerms; ++u) {
      if (chunks[u] <= 0) continue;
      add4(s, p[u]);
      if (chunks[u] > 1) {
        float4 q[kCompactMaxChunks];
#pragma unroll
        for (int c = 1; c < kCompactMaxChunks; ++c)
          if (c < chunks[u]) q[c] = partial[((int64_t)c * n_slots + slot[u]) * vecs + v];
#pragma unroll
        for (int c = 1; c < kCompactMaxChunks; ++c)
          if (c < chunks[u]) add4(s, q[c]);
      }
    }
  }
  Y[tok * vecs + v] = s;
}

// ---- work items and pairs of batches that the general counting sort puts in order -------------------------------
// The work items where the bucket order comes from the general counting sort.
__global__ __launch_bounds__(CAMERA_MAX_EXPERTS) void compact_items_kernel(CompactWork tab, int total,
                                                                           const int32_t* __restrict__ counts,
                                                                           int32_t* __restrict__ work) {
  __shared__ int32_t wave_total[CAMERA_MAX_EXPERTS / kWave];
  const int e = threadIdx.x;
  write_work<CAMERA_MAX_EXPERTS / kWave>(tab, total, e < total ? counts[e] : 0, wave_total, work);
}
// Where every expert has every token: the order too, in the one launch that the order alone would take.
__global__ __launch_bounds__(CAMERA_MAX_EXPERTS) void compact_dense_items_kernel(CompactWork tab, int total, int n,
                                                                                 int32_t* __restrict__ counts,
                                                                                 int32_t* __restrict__ offsets,
                                                                                 int32_t* __restrict__ work) {
  __shared__ int32_t wave_total[CAMERA_MAX_EXPERTS / kWave];
  const int e = threadIdx.x;
  if (e < total) {
    counts[e] = n;
    offsets[e] = e * n;
    if (e == total - 1) offsets[total] = total * n;
  }
  write_work<CAMERA_MAX_EXPERTS / kWave>(tab, total, e < total ? n : 0, wave_total, work);
}

// Upper bound of the work items of a contraction with tiles[e] per expert: of the n * top_k routed pairs, an expert with
// m of them has at most 1 + (m - 1) / 32 groups, so the first groups are at most one per expert (or pair) and the others
// one per 32 pairs; every appended (or dense) expert has all n tokens.  At most 2^22 workgroups (2^32 threads is the
// limit of a launch); they take further items in turn.
unsigned work_blocks(const int32_t* tiles, int n_routed, int total, int64_t n, int top_k) {
  int64_t sum = 0, widest = 0, all = 0;
  for (int e = 0; e < total; ++e) {
    if (e < n_routed) {
      sum += tiles[e];
      widest = widest > tiles[e] ? widest : tiles[e];
    } else {
      all += tiles[e] * ((n + kTokens - 1) / kTokens);
    }
  }
  const int64_t pairs = n * top_k;
  const int64_t first = sum < widest * pairs ? sum : widest * pairs;
  const int64_t blocks = first + widest * (pairs / kTokens) + all;
  return (unsigned)(blocks < (int64_t(1) << 22) ? blocks : (int64_t(1) << 22));
}

// The same pairs written out, for the general counting sort: idx_aug / w_aug [n][top_k + n_shared].
__global__ void compact_append_shared_kernel(const int32_t* __restrict__ topk_idx, const float* __restrict__ topk_w,
                                             int64_t n, int top_k, int n_experts, int n_shared,
                                             int32_t* __restrict__ idx_aug, float* __restrict__ w_aug) {
  const int kk = top_k + n_shared;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n * kk) return;
  const int64_t j = p / kk;
  const int k = (int)(p - j * kk);
  if (k < top_k) {
    const int e = topk_idx[j * top_k + k];
    idx_aug[p] = (e < 0 || e >= n_experts) ? -1 : e;  // an id of the appended experts is not a routed choice
    w_aug[p] = topk_w[j * top_k + k];
  } else {
    idx_aug[p] = n_experts + k - top_k;
    w_aug[p] = 1.0f;
  }
}

}  // namespace

hipError_t launch_compact_items(hipStream_t stream, const CompactWork& tab, int total, const BucketTables& t,
                                int32_t* work) {
  compact_items_kernel<<<1, CAMERA_MAX_EXPERTS, 0, stream>>>(tab, total, t.counts, work);
  return hipGetLastError();
}

hipError_t launch_compact_dense_items(hipStream_t stream, const CompactWork& tab, int total, int64_t n,
                                      const BucketTables& t, int32_t* work) {
  compact_dense_items_kernel<<<1, CAMERA_MAX_EXPERTS, 0, stream>>>(tab, total, (int)n, t.counts, t.offsets, work);
  return hipGetLastError();
}

hipError_t launch_compact_append_shared(hipStream_t stream, const int32_t* topk_idx, const float* topk_w, int64_t n,
                                        int top_k, int n_experts, int n_shared, int32_t* idx_aug, float* w_aug) {
  const int64_t pairs = n * (top_k + n_shared);
  compact_append_shared_kernel<<<(int)((pairs + 255) / 256), 256, 0, stream>>>(topk_idx, topk_w, n, top_k, n_experts,
                                                                                n_shared, idx_aug, w_aug);
  return hipGetLastError();
}

hipError_t launch_compact_hidden(hipStream_t stream, const void* X, int64_t ldx, int64_t d_model, const void* W_gate,
                                 const void* W_up, const CompactRows& tab, const CompactWork& tiles, int n_routed,
                                 int top_k, int64_t n, const BucketTables& t, const int32_t* work, void* hidden, int ldh) {
  const unsigned blocks = work_blocks(tiles.hidden_tiles, n_routed, tab.n_experts, n, top_k);
  if (blocks == 0) return hipSuccess;
  compact_hidden_kernel<kSplitHidden><<<blocks, kWave * kSplitHidden, 0, stream>>>(
      static_cast<const __bf16*>(X), ldx, (int)d_model, static_cast<const __bf16*>(W_gate),
      static_cast<const __bf16*>(W_up), tab, work, t.counts, t.offsets, t.perm, t.w_perm, static_cast<__bf16*>(hidden),
      ldh);
  return hipGetLastError();
}

hipError_t launch_compact_down(hipStream_t stream, const void* hidden, int ldh, const void* W_down, int64_t d_model,
                               const CompactDown& tab, const CompactWork& tiles, int n_routed, int top_k, int64_t n,
                               const BucketTables& t, const int32_t* work, int64_t n_slots, float* partial) {
  const unsigned blocks = work_blocks(tiles.down_tiles, n_routed, tab.n_experts, n, top_k);
  if (blocks == 0) return hipSuccess;
  work += CAMERA_MAX_EXPERTS + 1;
  int64_t kept = 0;
  for (int e = 0; e < tab.n_experts; ++e) kept += tab.count[e];
  if (kept >= (int64_t)kDownFourWavesFrom * tab.chunk_off[tab.n_experts])  // mean chunk length
    compact_down_kernel<4><<<blocks, kWave * 4, 0, stream>>>(static_cast<const __bf16*>(hidden), ldh,
                                                             static_cast<const __bf16*>(W_down), (int)d_model, tab, work,
                                                             t.counts, t.offsets, n_slots, partial);
  else
    compact_down_kernel<2><<<blocks, kWave * 2, 0, stream>>>(static_cast<const __bf16*>(hidden), ldh,
                                                             static_cast<const __bf16*>(W_down), (int)d_model, tab, work,
                                                             t.counts, t.offsets, n_slots, partial);
  return hipGetLastError();
}

hipError_t launch_compact_combine(hipStream_t stream, const float* partial, const CompactDown& tab,
                                  const BucketTables& t, const int32_t* topk_idx, int64_t n, int terms, int top_k,
                                  int n_routed, int64_t d_model, int64_t n_slots, int accumulate, float* Y) {
  const int vecs = (int)(d_model / 4);
  const int threads = vecs < 256 ? (vecs + kWave - 1) / kWave * kWave : 256;
  compact_combine_kernel<<<dim3((unsigned)n, (unsigned)((vecs + threads - 1) / threads)), threads, 0, stream>>>(
      reinterpret_cast<const float4*>(partial), t.slot_of, topk_idx, tab, n, terms, top_k, n_routed, vecs, n_slots,
      accumulate, reinterpret_cast<float4*>(Y));
  return hipGetLastError();
}

}  // namespace camera
