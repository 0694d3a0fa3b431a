// Ranking decisions on a layer's energies (Algorithm 1 line 11, Algorithm 2
// line 9, Algorithm 3 lines 5-8).  All integer work on float32 bit patterns.
//
// The order is the stable ascending order of (energy, index).  A cut at rank t
// separates the t lowest-ranked micro-experts from the rest; CAMERA-P needs one
// cut (t = n_prune), CAMERA-Q one per class boundary.  No sort is needed for
// that: a radix select (16 + 16 bits) finds, for every cut, the key K of the
// element of rank t and how many elements equal to K lie below the cut (r);
// element i is below the cut iff key_i < K, or key_i == K and fewer than r equal
// keys precede it.  The "equal keys that precede" count comes from an ordered
// walk: every wave owns a contiguous index range, ballots + popcounts give the
// order inside 64-element steps.
//
// rank_top / rank_low / rank_segment: all cuts of a call at once (the CAMERA-P
// cuts of several ratios and the CAMERA-Q class boundaries of a layer are cuts
// on the same order, so one set of passes serves both decisions).
// full rank: LSD radix sort (4 x 8 bits) of (key, index) built from a stable
// counting sort whose in-wave order again comes from ballots.
#include "camera_internal.h"

namespace camera {
namespace {

constexpr int kMaxCuts = CAMERA_MAX_LEVELS - 1;

__device__ __forceinline__ uint32_t key_of(float v) {
  uint32_t u = __float_as_uint(v);
  if (u == 0x80000000u) u = 0u;  // -0.0 ranks as +0.0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ---------------------------------------------------------------------------
// The decisions: two histogram passes over the keys, then the walk over the segments (experts).
//
// A layer has at most a few hundred thousand keys (<= 0.74 MB), so a call is bound by launches and by the latency of
// what each of them does in sequence, not by bandwidth.  Hence few passes and nothing serial between them:
//   top      one histogram of the upper 16 key bits, counted per workgroup in LDS (2^16 counters of 16 bits, 128 KiB)
//            and added to global memory where it is not zero: 8192 keys fall on one to two thousand values, so few
//            atomics leave a workgroup
//   low      the lower 16 bits of the keys that share a cut's upper 16; few keys do (a value of the upper 16 bits spans
//            1/128 of an octave), so they go to global memory one by one
//   segment  one workgroup per segment: class of every element, output bytes, counts and the stable partition by level
//   compact  (optional) ascending list of the kept indices
//   label, finish   instead of these two where a segment is long: a workgroup per part of one
// No workgroup picks for the others: `low` and `segment` begin with every workgroup reading the histogram of the pass
// before for itself -- a wave per cut, 256 coarse counters (8 bits) and then the 256 fine ones under the bin it found,
// two dependent loads -- so nothing needs a fence, a ticket or a last workgroup, and a kernel boundary is the only
// synchronisation.  Measured for 98 304 keys and five cuts: 26 us in 3 launches (7 + 10 + 9); with three passes of
// 11 + 11 + 10 bits over all keys and all cuts, each closed by a last workgroup that picked, 82 us in 5 launches, 53 of
// them in two passes' atomics and picks.  A call on 4096 keys: 18 us against 61.
// The select state cleans itself: it starts as zeros (the library clears it when it makes it), `top` clears what `low`
// will count in, `segment` clears what `top` counted in.  A call needs no clearing launch and leaves the state as it
// found it.  Equal keys that a cut runs through (energies of experts without tokens) are ordered by index inside the
// segment kernel, each workgroup counting the equal keys that precede it.
// ---------------------------------------------------------------------------
constexpr int kRankThreads = 1024;
constexpr int kRankWaves = kRankThreads / kWave;
constexpr int kKeysPerBlock = kRankThreads * 8;  // a counter of the LDS histogram cannot overflow its 16 bits
constexpr int kFine = 1 << 16, kCoarse = 1 << 8;
constexpr int kMaxParts = CAMERA_MAX_SEGMENTS + 1024;
constexpr int kMinTopBlocks = 64;                // workgroups that clear for `low` (0.25 MB per cut) when the keys are few
static_assert(kMaxCuts <= kRankWaves, "a wave per cut in the pick");

struct RankState {  // persistent, see above
  uint32_t top_coarse[kCoarse];           // counts by key bits 31..24
  uint32_t top_fine[kFine];               // counts by key bits 31..16
  struct Low {
    uint32_t coarse[kCoarse];             // of the keys that share the cut's bits 31..16: counts by bits 15..8
    uint32_t fine[kFine];                 // and by bits 15..0
  } low[kMaxCuts];
  uint32_t prefix[kMaxCuts];              // bits 31..16 of the cut element
  uint32_t rest[kMaxCuts];                // its rank among the keys that share them
  uint32_t part_class[kMaxParts][CAMERA_MAX_LEVELS];  // of a part of a segment: its members by class (written by `label`)
  uint32_t part_ties[kMaxParts][kMaxCuts];            // and the keys before it that equal each cut's, where a cut has ties
};

// The 8 keys of this thread: two float4 of consecutive keys, kKeysPerBlock / 2 apart.  Both loads are issued together.
struct Keys8 {
  uint32_t k[8];
  int n_valid[2];  // of each four, the valid ones come first
};
__device__ __forceinline__ Keys8 load_keys8(const float* __restrict__ E, int64_t n) {
  Keys8 out;
  float4 v[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kKeysPerBlock + u * (kKeysPerBlock / 2) + threadIdx.x * 4;
    out.n_valid[u] = i >= n ? 0 : (int)min((int64_t)4, n - i);
    if (out.n_valid[u] == 4) {
      v[u] = *reinterpret_cast<const float4*>(E + i);
    } else {
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (out.n_valid[u] > 0) v[u].x = E[i];
      if (out.n_valid[u] > 1) v[u].y = E[i + 1];
      if (out.n_valid[u] > 2) v[u].z = E[i + 2];
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    out.k[4 * u] = key_of(v[u].x);
    out.k[4 * u + 1] = key_of(v[u].y);
    out.k[4 * u + 2] = key_of(v[u].z);
    out.k[4 * u + 3] = key_of(v[u].w);
  }
  return out;
}

// A cut needs a select unless nothing or everything lies below it.
enum { kCutSelect = 0, kCutNone = 1, kCutAll = 2 };
__host__ __device__ inline int cut_mode(const RankCuts& cuts, int q, int64_t n) {
  if (q >= cuts.n_cuts || cuts.cut_rank[q] <= 0) return kCutNone;
  return cuts.cut_rank[q] >= n ? kCutAll : kCutSelect;
}

// By one whole wave: which of 256 counters holds the element of rank `rank`, and its rank inside that counter.
struct Pick {
  uint32_t bin, rest;
};
__device__ __forceinline__ Pick pick256(const uint32_t* __restrict__ counters, uint32_t rank) {
  const int lane = threadIdx.x % kWave;
  const uint4 c = *reinterpret_cast<const uint4*>(counters + lane * 4);
  const uint32_t sum = c.x + c.y + c.z + c.w;
  uint32_t before = sum;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t o = __shfl_up(before, d);
    if (lane >= d) before += o;
  }
  before -= sum;
  uint32_t bin = lane * 4, rest = rank - before;
  const bool mine = rank >= before && rest < sum;
  if (rest >= c.x) {
    rest -= c.x;
    ++bin;
    if (rest >= c.y) {
      rest -= c.y;
      ++bin;
      if (rest >= c.z) {
        rest -= c.z;
        ++bin;
      }
    }
  }
  const uint64_t who = __ballot(mine);
  const int src = who ? __ffsll((unsigned long long)who) - 1 : 0;  // exactly one lane: the counters add up to more than `rank`
  return {__shfl(bin, src), __shfl(rest, src)};
}
__device__ __forceinline__ Pick pick_2level(const uint32_t* coarse, const uint32_t* fine, uint32_t rank) {
  const Pick c = pick256(coarse, rank);
  const Pick f = pick256(fine + c.bin * kCoarse, c.rest);
  return {c.bin * kCoarse + f.bin, f.rest};
}

__global__ __launch_bounds__(kRankThreads) void rank_top_kernel(const float* __restrict__ E, int64_t n, int key_blocks,
                                                                int n_cuts, RankState* __restrict__ st) {
  __shared__ __align__(16) uint32_t hist[kFine / 2];  // pairs of 16-bit counters
  __shared__ uint32_t coarse[kCoarse];
  const int tid = threadIdx.x;
  const bool has_keys = (int)blockIdx.x < key_blocks;
  Keys8 keys;
  if (has_keys) keys = load_keys8(E, n);
  {  // this workgroup's share of the counters that `low` adds to: consecutive cuts are consecutive in memory
    uint4* low = reinterpret_cast<uint4*>(&st->low[0]);
    const int total = n_cuts * (int)(sizeof(RankState::Low) / 16);
    for (int i = blockIdx.x * kRankThreads + tid; i < total; i += gridDim.x * kRankThreads) low[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (!has_keys) return;  // block-uniform
#pragma unroll
  for (int i = 0; i < kFine / 8 / kRankThreads; ++i) reinterpret_cast<uint4*>(hist)[tid + i * kRankThreads] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < kCoarse) coarse[tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < keys.n_valid[u]) {
        const uint32_t top = keys.k[4 * u + j] >> 16;
        atomicAdd(&hist[top >> 1], 1u << (16 * (top & 1)));
      }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kFine / 8 / kRankThreads; ++i) {
    const int at = tid + i * kRankThreads;  // eight counters, all under one coarse one
    const uint4 c = reinterpret_cast<const uint4*>(hist)[at];
    if ((c.x | c.y | c.z | c.w) == 0u) continue;
    const uint32_t w[4] = {c.x, c.y, c.z, c.w};
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t lo = w[j] & 0xffffu, hi = w[j] >> 16;
      if (lo) atomicAdd(&st->top_fine[at * 8 + 2 * j], lo);
      if (hi) atomicAdd(&st->top_fine[at * 8 + 2 * j + 1], hi);
      sum += lo + hi;
    }
    atomicAdd(&coarse[at / (kCoarse / 8)], sum);
  }
  __syncthreads();
  if (tid < kCoarse && coarse[tid]) atomicAdd(&st->top_coarse[tid], coarse[tid]);
}

__global__ __launch_bounds__(kRankThreads) void rank_low_kernel(const float* __restrict__ E, int64_t n, RankCuts cuts,
                                                                RankState* __restrict__ st) {
  __shared__ uint32_t s_prefix[kMaxCuts];
  __shared__ uint32_t s_coarse[kMaxCuts][kCoarse];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const Keys8 keys = load_keys8(E, n);
  for (int i = tid; i < kMaxCuts * kCoarse; i += kRankThreads) (&s_coarse[0][0])[i] = 0u;
  if (wave < kMaxCuts) {
    Pick p = {0xffffffffu, 0u};  // not a value of 16 bits: no key matches
    if (cut_mode(cuts, wave, n) == kCutSelect) p = pick_2level(st->top_coarse, st->top_fine, (uint32_t)cuts.cut_rank[wave]);
    if (lane == 0) {
      s_prefix[wave] = p.bin;
      if (blockIdx.x == 0) {
        st->prefix[wave] = p.bin;
        st->rest[wave] = p.rest;
      }
    }
  }
  __syncthreads();
  uint32_t want[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) want[q] = s_prefix[q];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool valid = j < keys.n_valid[u];
      const uint32_t k = keys.k[4 * u + j], low = k & 0xffffu;
#pragma unroll
      for (int q = 0; q < kMaxCuts; ++q) {
        bool match = valid && (k >> 16) == want[q];
        uint64_t m = __ballot(match);
        if (m == 0) continue;  // wave-uniform
        if (match) atomicAdd(&s_coarse[q][low >> 8], 1u);
        // Many matches in one wave are mostly equal keys (experts without tokens): one addition for all that equal the
        // first, a few times; the rest, and the usual one or two, each for itself.
        for (int round = 0; round < 3 && __popcll(m) > 4; ++round) {
          const int leader = __ffsll((unsigned long long)m) - 1;
          const uint64_t same = __ballot(match && low == __shfl(low, leader));
          if (lane == leader) atomicAdd(&st->low[q].fine[low], (uint32_t)__popcll(same));
          m &= ~same;
          match = match && ((same >> lane) & 1) == 0;
        }
        if (match) atomicAdd(&st->low[q].fine[low], 1u);
      }
    }
  __syncthreads();
  for (int i = tid; i < kMaxCuts * kCoarse; i += kRankThreads) {
    const uint32_t c = (&s_coarse[0][0])[i];
    if (c) atomicAdd(&st->low[i / kCoarse].coarse[i % kCoarse], c);
  }
}

__device__ __forceinline__ int nibble(uint32_t packed, int c) { return (int)((packed >> (4 * c)) & 15u); }

// A segment of more keys than this goes in parts of kPartKeys or more: one workgroup walks some 1300 keys a microsecond, the
// parts cost a launch and, with a partition, two more walks.  us per call, whole / in parts (one pruning mask with its index
// list; three masks and bits; bits and partition):
//   64 segments of 2560, one of 20480   33 / 32    30 / 28    37 / 44
//   one of 32768                        39 / 28    34 / 24    45 / 41
//   one of 2^20                         802 / 54   563 / 48   992 / 65
constexpr int kWholeSegment = 24576;
constexpr int kPartKeys = 8192;

// The cuts as the walk sees them.
struct CutKeys {
  uint32_t key[kMaxCuts];   // key of the cut element; 0, which no key is below, where nothing or everything lies below
  uint32_t ties[kMaxCuts];  // how many keys equal to it lie below the cut
  uint32_t all;             // bit q: everything lies below cut q
};

// Number of cuts that the element with key k is below.  tie_run[q]: keys equal to the cut's at lower indices than this
// wave's step; moved on by the step.  ANY_TIES: some cut runs through a group of equal keys.
template <bool ANY_TIES>
__device__ __forceinline__ int class_of(const CutKeys& c, uint32_t k, bool valid, uint64_t lower, uint32_t* tie_run) {
  int below = __popc(c.all);
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) {
    below += k < c.key[q] ? 1 : 0;
    if (ANY_TIES && c.ties[q] != 0) {  // block-uniform
      const bool eq = valid && k == c.key[q];
      const uint64_t b = __ballot(eq);
      if (eq && tie_run[q] + __popcll(b & lower) < c.ties[q]) below += 1;
      tie_run[q] += __popcll(b);
    }
  }
  return below;
}

// A wave's range of [begin, end): the waves have consecutive ones, whole steps of kWave.
struct WaveRange {
  int begin, end;
};
__device__ __forceinline__ WaveRange wave_range(int begin, int end) {
  const int wave = threadIdx.x / kWave;
  const int span = ((end - begin + kRankWaves * kWave - 1) / (kRankWaves * kWave)) * kWave;
  WaveRange r;
  r.begin = min(end, begin + wave * span);
  r.end = min(end, r.begin + span);
  return r;
}
constexpr int kSteps = 4;  // steps of a walk whose loads are in flight together

// A cut runs through equal keys in one call of ten or so (two adjacent keys of 180 000 are equal with a chance of 2 %): those
// before a segment are counted with 16-byte loads, four in flight per thread (one mask of 64 segments of 2560 and one of 20480
// with one such pair: 56 us, with 4-byte loads and every cut compared 89, without a tie 33).
// tie_base[q]: keys equal to cut q's at lower indices than the wave's range, where the cut has ties.  COUNT_BEFORE: those
// before `begin` are counted here, by all threads, and left in s_before (all of the workgroup's waves call it); otherwise
// s_before has them.
template <bool COUNT_BEFORE>
__device__ __forceinline__ void count_ties(const float* __restrict__ E, const CutKeys& cut, int begin, WaveRange r,
                                           uint32_t* s_before, uint32_t (*s_tie)[kRankWaves], uint32_t (&tie_base)[kMaxCuts]) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  uint32_t before[kMaxCuts], mine[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) before[q] = mine[q] = 0u;
  // Only cuts that run through equal keys are counted (block-uniform): with more it is the comparisons that take the time.
  if constexpr (COUNT_BEFORE) {
    constexpr int U = kSteps;
    const int64_t vecs = begin / 4;  // E is 16-byte aligned
    for (int64_t i0 = threadIdx.x; i0 < vecs; i0 += U * kRankThreads) {  // 64 bits: an index may be within a step of 2^31
      uint4 k[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float4 v = reinterpret_cast<const float4*>(E)[min(i0 + u * kRankThreads, vecs - 1)];
        k[u] = make_uint4(key_of(v.x), key_of(v.y), key_of(v.z), key_of(v.w));
      }
#pragma unroll
      for (int q = 0; q < kMaxCuts; ++q) {
        if (cut.ties[q] == 0) continue;
        const uint32_t want = cut.key[q];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * kRankThreads < vecs)
            before[q] += (k[u].x == want ? 1u : 0u) + (k[u].y == want ? 1u : 0u) + (k[u].z == want ? 1u : 0u) + (k[u].w == want ? 1u : 0u);
      }
    }
    const int64_t rest = vecs * 4 + threadIdx.x;
    if (rest < begin) {
      const uint32_t k = key_of(E[rest]);
#pragma unroll
      for (int q = 0; q < kMaxCuts; ++q) before[q] += cut.ties[q] != 0 && k == cut.key[q] ? 1u : 0u;
    }
  }
  for (int i0 = r.begin; i0 < r.end; i0 += kSteps * kWave) {
    float v[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) v[u] = E[min(i0 + u * kWave + lane, r.end - 1)];
#pragma unroll
    for (int q = 0; q < kMaxCuts; ++q) {
      if (cut.ties[q] == 0) continue;
#pragma unroll
      for (int u = 0; u < kSteps; ++u)
        mine[q] += __popcll(__ballot(i0 + u * kWave + lane < r.end && key_of(v[u]) == cut.key[q]));
    }
  }
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) {
    if constexpr (COUNT_BEFORE) {
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) before[q] += __shfl_xor(before[q], m);
    }
    if (lane == 0) {
      s_tie[q][wave] = mine[q];
      s_tie[kMaxCuts + q][wave] = before[q];
    }
  }
  __syncthreads();
  if (COUNT_BEFORE && threadIdx.x < kMaxCuts) {
    uint32_t all = 0;
    for (int w = 0; w < kRankWaves; ++w) all += s_tie[kMaxCuts + threadIdx.x][w];
    s_before[threadIdx.x] = all;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) {
    uint32_t run = s_before[q];
    for (int w = 0; w < wave; ++w) run += s_tie[q][w];
    tie_base[q] = run;
  }
}

// f(index, valid, class) for the elements of the wave's range, in index order, all lanes together.
template <bool ANY_TIES, class F>
__device__ __forceinline__ void walk(const float* __restrict__ E, const CutKeys& cut, WaveRange r,
                                     const uint32_t (&tie_base)[kMaxCuts], F&& f) {
  const int lane = threadIdx.x % kWave;
  const uint64_t lower = (1ull << lane) - 1ull;
  uint32_t tie_run[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) tie_run[q] = tie_base[q];
  for (int i0 = r.begin; i0 < r.end; i0 += kSteps * kWave) {
    float v[kSteps];
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const int i = i0 + u * kWave + lane;
      v[u] = i < r.end ? E[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kSteps; ++u) {
      const int i = i0 + u * kWave + lane;
      const bool valid = i < r.end;
      f(i, valid, class_of<ANY_TIES>(cut, key_of(v[u]), valid, lower, tie_run));
    }
  }
}

// The cuts' keys from the counts of the `low` pass, by every workgroup for itself.
__device__ __forceinline__ void load_cuts(const RankCuts& cuts, int64_t n, const RankState* __restrict__ st, uint32_t* s_key,
                                          uint32_t* s_ties, CutKeys* cut, bool* any_ties) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  if (wave < kMaxCuts) {
    Pick p = {0u, 0u};
    if (cut_mode(cuts, wave, n) == kCutSelect) {
      p = pick_2level(st->low[wave].coarse, st->low[wave].fine, st->rest[wave]);
      p.bin |= st->prefix[wave] << 16;
    }
    if (lane == 0) {
      s_key[wave] = p.bin;
      s_ties[wave] = p.rest;
    }
  }
  __syncthreads();
  cut->all = 0u;
  *any_ties = false;
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) {
    cut->key[q] = __builtin_amdgcn_readfirstlane(s_key[q]);
    cut->ties[q] = __builtin_amdgcn_readfirstlane(s_ties[q]);
    *any_ties |= cut->ties[q] != 0;
    if (cut_mode(cuts, q, n) == kCutAll) cut->all |= 1u << q;
  }
}
// Leaves the counters of the `top` pass as the next call needs them; nobody reads them any more.
__device__ __forceinline__ void clear_top(RankState* __restrict__ st) {
  uint4* top = reinterpret_cast<uint4*>(st->top_coarse);
  static_assert(offsetof(RankState, top_fine) == kCoarse * 4, "coarse and fine counters lie side by side");
  for (int i = blockIdx.x * kRankThreads + threadIdx.x; i < (kCoarse + kFine) / 4; i += gridDim.x * kRankThreads)
    top[i] = make_uint4(0u, 0u, 0u, 0u);
}
struct OutTables {
  uint64_t first, second;  // output bytes by class
};
__device__ __forceinline__ OutTables out_tables(const RankCuts& cuts) {
  OutTables t = {0, 0};
#pragma unroll
  for (int c = 0; c <= kMaxCuts; ++c) {
    t.first |= (uint64_t)cuts.out_of_below[c] << (8 * c);
    t.second |= (uint64_t)cuts.out2_of_below[c] << (8 * c);
  }
  return t;
}

// Output bytes of the wave's elements (WRITE); s_cnt[wave]: its members by class.
template <bool ANY_TIES, bool WRITE>
__device__ __forceinline__ void label(const float* __restrict__ E, const CutKeys& cut, WaveRange r,
                                      const uint32_t (&tie_base)[kMaxCuts], const OutTables& t, int n_classes,
                                      uint8_t* __restrict__ byte_out, uint8_t* __restrict__ byte_out2,
                                      uint32_t (*s_cnt)[CAMERA_MAX_LEVELS]) {
  uint32_t cnt[CAMERA_MAX_LEVELS];
#pragma unroll
  for (int m = 0; m < CAMERA_MAX_LEVELS; ++m) cnt[m] = 0u;
  walk<ANY_TIES>(E, cut, r, tie_base, [&](int i, bool valid, int c) {
    if (WRITE && valid) {
      byte_out[i] = (uint8_t)(t.first >> (8 * c));
      if (byte_out2) byte_out2[i] = (uint8_t)(t.second >> (8 * c));
    }
#pragma unroll
    for (int m = 0; m < CAMERA_MAX_LEVELS; ++m)
      if (m < n_classes) cnt[m] += __popcll(__ballot(valid && c == m));
  });
  if (threadIdx.x % kWave == 0) {
#pragma unroll
    for (int m = 0; m < CAMERA_MAX_LEVELS; ++m) s_cnt[threadIdx.x / kWave][m] = cnt[m];
  }
}
// Members of level m among the classes counted in cnt.
__device__ __forceinline__ uint32_t of_level(const SegOutputs& out, const uint32_t* cnt, int m) {
  uint32_t total = 0;
  for (int c = 0; c < out.n_classes; ++c)
    if (nibble(out.level_of_class, c) == m) total += cnt[c];
  return total;
}
// Kept at ratio k: the members of the classes that lie below at most n_ratios - 1 - k of the pruning cuts.
__device__ __forceinline__ bool class_kept(const SegOutputs& out, int c, int k) {
  return nibble(out.prune_cuts_of_class, c) <= out.n_ratios - 1 - k;
}
// The stable partition by level: slot[m] is the first place of the wave's members of level m.
template <bool ANY_TIES>
__device__ __forceinline__ void partition(const float* __restrict__ E, const CutKeys& cut, WaveRange r,
                                          const uint32_t (&tie_base)[kMaxCuts], const SegOutputs& out,
                                          uint32_t (&slot)[CAMERA_MAX_LEVELS]) {
  const uint64_t lower = (1ull << (threadIdx.x % kWave)) - 1ull;
  walk<ANY_TIES>(E, cut, r, tie_base, [&](int i, bool valid, int c) {
    const int lv = nibble(out.level_of_class, c);
#pragma unroll
    for (int m = 0; m < CAMERA_MAX_LEVELS; ++m) {
      if (m < out.n_levels) {
        const uint64_t b = __ballot(valid && lv == m);
        if (valid && lv == m) out.perm[slot[m] + __popcll(b & lower)] = i;
        slot[m] += __popcll(b);
      }
    }
  });
}

// One workgroup per segment.  low_counted: the select passes ran (some cut has keys on both sides).
template <bool ANY_TIES>
__device__ __forceinline__ void whole_segment(const float* __restrict__ E, const CutKeys& cut, int begin, int end,
                                              const OutTables& t, const SegOutputs& out, int n_seg,
                                              uint8_t* __restrict__ byte_out, uint8_t* __restrict__ byte_out2,
                                              uint32_t (*s_cnt)[CAMERA_MAX_LEVELS], uint32_t (*s_lvl)[CAMERA_MAX_LEVELS],
                                              uint32_t (*s_tie)[kRankWaves], uint32_t* s_before) {
  const int s = blockIdx.x, wave = threadIdx.x / kWave;
  const WaveRange r = wave_range(begin, end);
  uint32_t tie_base[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) tie_base[q] = 0u;
  if constexpr (ANY_TIES) count_ties<true>(E, cut, begin, r, s_before, s_tie, tie_base);
  label<ANY_TIES, true>(E, cut, r, tie_base, t, out.n_classes, byte_out, byte_out2, s_cnt);
  __syncthreads();
  if (threadIdx.x < kRankWaves * CAMERA_MAX_LEVELS) {  // (wave w, level m): members of level m in wave w's range
    const int w = threadIdx.x / CAMERA_MAX_LEVELS, m = threadIdx.x % CAMERA_MAX_LEVELS;
    s_lvl[w][m] = of_level(out, s_cnt[w], m);
  }
  if (threadIdx.x >= 512 && threadIdx.x < 512 + out.n_ratios) {
    const int k = threadIdx.x - 512;
    uint32_t total = 0;
    for (int c = 0; c < out.n_classes; ++c)
      if (class_kept(out, c, k))
        for (int w = 0; w < kRankWaves; ++w) total += s_cnt[w][c];
    out.kept[k * n_seg + s] = (int32_t)total;
  }
  __syncthreads();
  if (threadIdx.x < out.n_levels) {
    uint32_t total = 0;
    for (int w = 0; w < kRankWaves; ++w) total += s_lvl[w][threadIdx.x];
    out.level_count[s * out.n_levels + threadIdx.x] = (int32_t)total;
  }
  if (out.perm == nullptr) return;  // block-uniform
  // first slot of level m for this wave = segment start + all earlier levels + earlier waves
  uint32_t slot[CAMERA_MAX_LEVELS];
  uint32_t run = (uint32_t)begin;
#pragma unroll
  for (int m = 0; m < CAMERA_MAX_LEVELS; ++m) {
    slot[m] = 0;
    if (m < out.n_levels) {
      for (int w = 0; w < kRankWaves; ++w) {
        if (w == wave) slot[m] = run;
        run += s_lvl[w][m];
      }
    }
  }
  partition<ANY_TIES>(E, cut, r, tie_base, out, slot);
}

__global__ __launch_bounds__(kRankThreads) void rank_segment_kernel(const float* __restrict__ E, int64_t n, RankCuts cuts,
                                                                   SegTable seg, SegOutputs out, int low_counted,
                                                                   RankState* __restrict__ st, uint8_t* __restrict__ byte_out,
                                                                   uint8_t* __restrict__ byte_out2 /*or NULL*/) {
  __shared__ uint32_t s_key[kMaxCuts], s_ties[kMaxCuts], s_before[kMaxCuts];
  __shared__ uint32_t s_cnt[kRankWaves][CAMERA_MAX_LEVELS];   // per wave and class
  __shared__ uint32_t s_lvl[kRankWaves][CAMERA_MAX_LEVELS];   // per wave and level
  __shared__ uint32_t s_tie[2 * kMaxCuts][kRankWaves];
  if (low_counted) clear_top(st);
  CutKeys cut;
  bool any_ties;
  load_cuts(cuts, n, st, s_key, s_ties, &cut, &any_ties);
  const OutTables t = out_tables(cuts);
  const int begin = seg.off[blockIdx.x], end = seg.off[blockIdx.x + 1];
  if (any_ties)  // block-uniform
    whole_segment<true>(E, cut, begin, end, t, out, seg.n_seg, byte_out, byte_out2, s_cnt, s_lvl, s_tie, s_before);
  else
    whole_segment<false>(E, cut, begin, end, t, out, seg.n_seg, byte_out, byte_out2, s_cnt, s_lvl, s_tie, s_before);
}

// Long segments go in parts of `len` keys, a workgroup each, in two launches: `label` writes the output bytes and counts a
// part's members by class, `finish` adds the parts up and places their members.  off[s]: the parts before segment s; a
// segment without keys has one part.
struct Parts {
  int32_t len;
  uint16_t off[CAMERA_MAX_SEGMENTS + 1];
};
static_assert(kMaxParts < 65536, "part numbers fit 16 bits");
struct PartRange {
  int seg, begin, end;
};
__device__ __forceinline__ PartRange part_range(const Parts& parts, const SegTable& seg, int* s_seg) {
  const int b = blockIdx.x;
  if ((int)threadIdx.x < seg.n_seg && parts.off[threadIdx.x] <= b && b < parts.off[threadIdx.x + 1]) *s_seg = threadIdx.x;
  __syncthreads();
  PartRange p;
  p.seg = __builtin_amdgcn_readfirstlane(*s_seg);
  const int64_t begin = seg.off[p.seg] + (int64_t)(b - parts.off[p.seg]) * parts.len;
  p.begin = (int)begin;
  p.end = (int)min(begin + parts.len, (int64_t)seg.off[p.seg + 1]);
  return p;
}

__global__ __launch_bounds__(kRankThreads) void rank_label_kernel(const float* __restrict__ E, int64_t n, RankCuts cuts,
                                                                 SegTable seg, Parts parts, int n_classes, int low_counted,
                                                                 RankState* __restrict__ st, uint8_t* __restrict__ byte_out,
                                                                 uint8_t* __restrict__ byte_out2 /*or NULL*/) {
  __shared__ uint32_t s_key[kMaxCuts], s_ties[kMaxCuts], s_before[kMaxCuts];
  __shared__ uint32_t s_cnt[kRankWaves][CAMERA_MAX_LEVELS];
  __shared__ uint32_t s_tie[2 * kMaxCuts][kRankWaves];
  __shared__ int s_seg;
  if (low_counted) clear_top(st);
  const PartRange p = part_range(parts, seg, &s_seg);
  CutKeys cut;
  bool any_ties;
  load_cuts(cuts, n, st, s_key, s_ties, &cut, &any_ties);
  const OutTables t = out_tables(cuts);
  const WaveRange r = wave_range(p.begin, p.end);
  uint32_t tie_base[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) tie_base[q] = 0u;
  if (any_ties) {  // block-uniform
    count_ties<true>(E, cut, p.begin, r, s_before, s_tie, tie_base);
    if (threadIdx.x < kMaxCuts) st->part_ties[blockIdx.x][threadIdx.x] = s_before[threadIdx.x];
    label<true, true>(E, cut, r, tie_base, t, n_classes, byte_out, byte_out2, s_cnt);
  } else {
    label<false, true>(E, cut, r, tie_base, t, n_classes, byte_out, byte_out2, s_cnt);
  }
  __syncthreads();
  if (threadIdx.x < CAMERA_MAX_LEVELS) {
    uint32_t total = 0;
    for (int w = 0; w < kRankWaves; ++w) total += s_cnt[w][threadIdx.x];
    st->part_class[blockIdx.x][threadIdx.x] = total;
  }
}

// kept_idx as in rank_compact_kernel.
template <bool ANY_TIES>
__device__ __forceinline__ void place_part(const float* __restrict__ E, const CutKeys& cut, const PartRange& p,
                                           const SegOutputs& out, const uint32_t* s_total, const uint32_t* s_earlier,
                                           uint32_t first_kept, int32_t* __restrict__ kept_idx,
                                           uint32_t (*s_cnt)[CAMERA_MAX_LEVELS], uint32_t (*s_tie)[kRankWaves],
                                           uint32_t* s_before, int seg_begin) {
  const int wave = threadIdx.x / kWave;
  const uint64_t lower = (1ull << (threadIdx.x % kWave)) - 1ull;
  const WaveRange r = wave_range(p.begin, p.end);
  uint32_t tie_base[kMaxCuts];
#pragma unroll
  for (int q = 0; q < kMaxCuts; ++q) tie_base[q] = 0u;
  if constexpr (ANY_TIES) count_ties<false>(E, cut, p.begin, r, s_before, s_tie, tie_base);
  label<ANY_TIES, false>(E, cut, r, tie_base, OutTables{0, 0}, out.n_classes, nullptr, nullptr, s_cnt);
  __syncthreads();
  if (out.perm) {
    uint32_t slot[CAMERA_MAX_LEVELS];
    uint32_t run = (uint32_t)seg_begin;
#pragma unroll
    for (int m = 0; m < CAMERA_MAX_LEVELS; ++m) {
      slot[m] = 0;
      if (m < out.n_levels) {
        slot[m] = run + of_level(out, s_earlier, m);
        for (int w = 0; w < wave; ++w) slot[m] += of_level(out, s_cnt[w], m);
        run += of_level(out, s_total, m);
      }
    }
    partition<ANY_TIES>(E, cut, r, tie_base, out, slot);
  }
  if (kept_idx) {
    uint32_t pos = first_kept;
    for (int w = 0; w < wave; ++w) pos += s_cnt[w][0];
    walk<ANY_TIES>(E, cut, r, tie_base, [&](int i, bool valid, int c) {
      const uint64_t b = __ballot(valid && c == 0);
      if (valid && c == 0) kept_idx[pos + __popcll(b & lower)] = i;
      pos += __popcll(b);
    });
  }
}

__global__ __launch_bounds__(kRankThreads) void rank_finish_kernel(const float* __restrict__ E, int64_t n, RankCuts cuts,
                                                                  SegTable seg, Parts parts, SegOutputs out,
                                                                  const RankState* __restrict__ st,
                                                                  int32_t* __restrict__ kept_idx /*or NULL*/) {
  __shared__ uint32_t s_key[kMaxCuts], s_ties[kMaxCuts], s_before[kMaxCuts];
  __shared__ uint32_t s_cnt[kRankWaves][CAMERA_MAX_LEVELS];
  __shared__ uint32_t s_tie[2 * kMaxCuts][kRankWaves];
  __shared__ uint32_t s_total[CAMERA_MAX_LEVELS], s_earlier[CAMERA_MAX_LEVELS];  // of the segment, of its earlier parts
  __shared__ uint32_t s_kept;                                                    // before this part, in all segments
  __shared__ int s_seg;
  const int b = blockIdx.x, tid = threadIdx.x;
  if (tid < CAMERA_MAX_LEVELS) s_total[tid] = s_earlier[tid] = 0u;
  if (tid == 0) s_kept = 0u;
  const PartRange p = part_range(parts, seg, &s_seg);
  for (int i = parts.off[p.seg] + tid / CAMERA_MAX_LEVELS; i < parts.off[p.seg + 1]; i += kRankThreads / CAMERA_MAX_LEVELS) {
    const int c = tid % CAMERA_MAX_LEVELS;
    const uint32_t v = st->part_class[i][c];
    if (v == 0u) continue;
    atomicAdd(&s_total[c], v);
    if (i < b) atomicAdd(&s_earlier[c], v);
  }
  if (kept_idx) {
    for (int i = tid; i < b; i += kRankThreads) atomicAdd(&s_kept, st->part_class[i][0]);
  }
  if (tid < kMaxCuts) s_before[tid] = st->part_ties[b][tid];
  CutKeys cut;
  bool any_ties;
  load_cuts(cuts, n, st, s_key, s_ties, &cut, &any_ties);
  if (b == parts.off[p.seg]) {
    if (tid < out.n_ratios) {
      uint32_t total = 0;
      for (int c = 0; c < out.n_classes; ++c) total += class_kept(out, c, tid) ? s_total[c] : 0u;
      out.kept[tid * seg.n_seg + p.seg] = (int32_t)total;
    }
    if (tid < out.n_levels) out.level_count[p.seg * out.n_levels + tid] = (int32_t)of_level(out, s_total, tid);
  }
  if (out.perm == nullptr && kept_idx == nullptr) return;  // block-uniform
  if (any_ties)  // block-uniform
    place_part<true>(E, cut, p, out, s_total, s_earlier, s_kept, kept_idx, s_cnt, s_tie, s_before, seg.off[p.seg]);
  else
    place_part<false>(E, cut, p, out, s_total, s_earlier, s_kept, kept_idx, s_cnt, s_tie, s_before, seg.off[p.seg]);
}

// Ascending list of the kept indices (keep byte 1), one workgroup per segment; kept [n_seg]: how many each segment keeps.
__global__ __launch_bounds__(kRankThreads) void rank_compact_kernel(const uint8_t* __restrict__ keep, SegTable seg,
                                                                   const int32_t* __restrict__ kept,
                                                                   int32_t* __restrict__ kept_idx) {
  __shared__ uint32_t s_first, s_mine[kRankWaves];
  const int s = blockIdx.x, lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const uint64_t lower = (1ull << lane) - 1ull;
  const int begin = seg.off[s], end = seg.off[s + 1];
  const int span = ((end - begin + kRankWaves * kWave - 1) / (kRankWaves * kWave)) * kWave;
  const int w_begin = min(end, begin + wave * span);
  const int w_end = min(end, w_begin + span);
  constexpr int U = 4;
  if (wave == 0) {
    uint32_t first = 0;
    for (int b = lane; b < s; b += kWave) first += (uint32_t)kept[b];
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) first += __shfl_xor(first, m);
    if (lane == 0) s_first = first;
  }
  auto walk = [&](auto&& step) {  // step(index, kept) in index order, all lanes together
    for (int i0 = w_begin; i0 < w_end; i0 += U * kWave) {
      uint8_t b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * kWave + lane;
        b[u] = i < w_end ? keep[i] : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) step(i0 + u * kWave + lane, b[u] != 0);
    }
  };
  uint32_t mine = 0;
  walk([&](int, bool k) { mine += __popcll(__ballot(k)); });
  if (lane == 0) s_mine[wave] = mine;
  __syncthreads();
  uint32_t pos = s_first;
  for (int w = 0; w < wave; ++w) pos += s_mine[w];
  walk([&](int i, bool k) {
    const uint64_t b = __ballot(k);
    if (k) kept_idx[pos + __popcll(b & lower)] = i;
    pos += __popcll(b);
  });
}

__global__ __launch_bounds__(kRankThreads) void rank_clear_kernel(uint4* __restrict__ state, int vecs) {
  for (int i = blockIdx.x * kRankThreads + threadIdx.x; i < vecs; i += gridDim.x * kRankThreads)
    state[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---------------------------------------------------------------------------
// full rank: LSD radix sort of (key, index), 8 bits per pass
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortChunk = 2048;                          // keys per block
constexpr int kSortPerWave = kSortChunk / kSortWaves;     // 512 consecutive keys per wave
constexpr int kDigits = 256;

__global__ __launch_bounds__(kSortThreads) void sort_init_kernel(const float* __restrict__ E, int64_t n,
                                                                 uint32_t* __restrict__ keys,
                                                                 uint32_t* __restrict__ idx) {
  const int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
  if (i < n) {
    keys[i] = key_of(E[i]);
    idx[i] = (uint32_t)i;
  }
}

__global__ __launch_bounds__(kSortThreads) void sort_count_kernel(const uint32_t* __restrict__ keys, int64_t n,
                                                                  int shift, int32_t* __restrict__ block_hist) {
  __shared__ int32_t hist[kDigits];
  hist[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortChunk;
  for (int i = threadIdx.x; i < kSortChunk; i += kSortThreads)
    if (base + i < n) atomicAdd(&hist[(keys[base + i] >> shift) & 0xff], 1);
  __syncthreads();
  block_hist[(int64_t)blockIdx.x * kDigits + threadIdx.x] = hist[threadIdx.x];
}

// one block; thread d owns digit d: exclusive bases over (digit, block)
__global__ __launch_bounds__(kDigits) void sort_scan_kernel(int32_t* __restrict__ block_hist, int n_blocks) {
  __shared__ int32_t s_total[kDigits];
  __shared__ int32_t s_base[kDigits];
  const int d = threadIdx.x;
  int32_t total = 0;
  for (int b = 0; b < n_blocks; ++b) {
    const int32_t c = block_hist[(int64_t)b * kDigits + d];
    block_hist[(int64_t)b * kDigits + d] = total;
    total += c;
  }
  s_total[d] = total;
  __syncthreads();
  if (d == 0) {
    int32_t run = 0;
    for (int i = 0; i < kDigits; ++i) {
      s_base[i] = run;
      run += s_total[i];
    }
  }
  __syncthreads();
  const int32_t base = s_base[d];
  for (int b = 0; b < n_blocks; ++b) block_hist[(int64_t)b * kDigits + d] += base;
}

// stable scatter; in the last pass the destination position is written to rank[idx]
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(const uint32_t* __restrict__ keys_in,
                                                                    const uint32_t* __restrict__ idx_in, int64_t n,
                                                                    int shift, const int32_t* __restrict__ block_base,
                                                                    uint32_t* __restrict__ keys_out,
                                                                    uint32_t* __restrict__ idx_out,
                                                                    uint32_t* __restrict__ rank_out) {
  __shared__ int32_t next[kSortWaves][kDigits];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t wave_first = (int64_t)blockIdx.x * kSortChunk + (int64_t)wave * kSortPerWave;
  for (int i = threadIdx.x; i < kSortWaves * kDigits; i += kSortThreads) (&next[0][0])[i] = 0;
  __syncthreads();
  for (int it = 0; it < kSortPerWave / kWave; ++it) {
    const int64_t p = wave_first + it * kWave + lane;
    if (p < n) atomicAdd(&next[wave][(keys_in[p] >> shift) & 0xff], 1);
  }
  __syncthreads();
  {
    const int d = threadIdx.x;  // kSortThreads == kDigits
    int32_t run = block_base[(int64_t)blockIdx.x * kDigits + d];
    for (int w = 0; w < kSortWaves; ++w) {
      const int32_t c = next[w][d];
      next[w][d] = run;
      run += c;
    }
  }
  __syncthreads();
  const uint64_t lower = (1ull << lane) - 1ull;
  for (int it = 0; it < kSortPerWave / kWave; ++it) {
    const int64_t p = wave_first + it * kWave + lane;
    int digit = -1;
    uint32_t key = 0, id = 0;
    if (p < n) {
      key = keys_in[p];
      id = idx_in[p];
      digit = (int)((key >> shift) & 0xff);
    }
    uint64_t waiting = __ballot(digit >= 0);
    int dst = -1;
    while (waiting) {
      const int leader = __ffsll((unsigned long long)waiting) - 1;
      const int ld = __shfl(digit, leader);
      const uint64_t same = __ballot(digit == ld);
      if (digit == ld) dst = next[wave][ld] + __popcll(same & lower);
      __builtin_amdgcn_wave_barrier();
      if (lane == leader) next[wave][ld] += __popcll(same);
      __builtin_amdgcn_wave_barrier();
      waiting &= ~same;
    }
    if (digit >= 0) {
      if (rank_out) {
        rank_out[id] = (uint32_t)dst;
      } else {
        keys_out[dst] = key;
        idx_out[dst] = id;
      }
    }
  }
}

static_assert(kSortThreads == kDigits, "one thread per digit in the scatter prologue");

}  // namespace

size_t rank_state_bytes() { return (sizeof(RankState) + 15) & ~size_t(15); }

hipError_t launch_rank_clear(hipStream_t stream, void* state) {
  hipLaunchKernelGGL(rank_clear_kernel, dim3(kMinTopBlocks), dim3(kRankThreads), 0, stream, static_cast<uint4*>(state),
                     (int)(rank_state_bytes() / 16));
  return hipGetLastError();
}

int64_t rank_workspace_words(int64_t n_micro, int want_rank) {
  if (!want_rank) return 0;
  const int64_t n_blocks = (n_micro + kSortChunk - 1) / kSortChunk;
  return 4 * (n_micro + 64) + n_blocks * kDigits;
}

hipError_t launch_rank_decisions(hipStream_t stream, const float* energy, int64_t n_micro, const RankCuts& cuts,
                                 const SegTable& seg, const SegOutputs& out, uint8_t* byte_out, uint8_t* byte_out2,
                                 int32_t* kept_idx, void* state) {
  RankState* st = static_cast<RankState*>(state);
  bool select = false;
  for (int q = 0; q < cuts.n_cuts; ++q) select |= cut_mode(cuts, q, n_micro) == kCutSelect;
  if (select) {
    const int blocks = (int)((n_micro + kKeysPerBlock - 1) / kKeysPerBlock);
    hipLaunchKernelGGL(rank_top_kernel, dim3((unsigned)(blocks > kMinTopBlocks ? blocks : kMinTopBlocks)), dim3(kRankThreads),
                       0, stream, energy, n_micro, blocks, cuts.n_cuts, st);
    hipLaunchKernelGGL(rank_low_kernel, dim3((unsigned)blocks), dim3(kRankThreads), 0, stream, energy, n_micro, cuts, st);
  }
  int widest = 0;
  for (int i = 0; i < seg.n_seg; ++i) widest = seg.off[i + 1] - seg.off[i] > widest ? seg.off[i + 1] - seg.off[i] : widest;
  if (widest <= kWholeSegment) {
    hipLaunchKernelGGL(rank_segment_kernel, dim3((unsigned)seg.n_seg), dim3(kRankThreads), 0, stream, energy, n_micro, cuts,
                       seg, out, select ? 1 : 0, st, byte_out, byte_out2);
    if (kept_idx && n_micro > 0)
      hipLaunchKernelGGL(rank_compact_kernel, dim3((unsigned)seg.n_seg), dim3(kRankThreads), 0, stream, byte_out, seg, out.kept,
                         kept_idx);
    return hipGetLastError();
  }
  Parts parts;
  const int64_t most = kMaxParts - CAMERA_MAX_SEGMENTS;  // a part begins at every segment and after `len` keys
  const int64_t len = ((n_micro + most - 1) / most + kRankThreads - 1) / kRankThreads * kRankThreads;
  parts.len = (int32_t)(len > kPartKeys ? len : kPartKeys);
  int n_parts = 0;
  for (int i = 0; i < seg.n_seg; ++i) {
    parts.off[i] = (uint16_t)n_parts;
    const int64_t keys = seg.off[i + 1] - seg.off[i];
    n_parts += keys > 0 ? (int)((keys + parts.len - 1) / parts.len) : 1;
  }
  for (int i = seg.n_seg; i <= CAMERA_MAX_SEGMENTS; ++i) parts.off[i] = (uint16_t)n_parts;
  hipLaunchKernelGGL(rank_label_kernel, dim3((unsigned)n_parts), dim3(kRankThreads), 0, stream, energy, n_micro, cuts, seg, parts,
                     out.n_classes, select ? 1 : 0, st, byte_out, byte_out2);
  hipLaunchKernelGGL(rank_finish_kernel, dim3((unsigned)n_parts), dim3(kRankThreads), 0, stream, energy, n_micro, cuts, seg,
                     parts, out, st, kept_idx);
  return hipGetLastError();
}

hipError_t launch_full_rank(hipStream_t stream, const float* energy, int64_t n_micro, uint32_t* rank,
                            int32_t* ws) {
  if (n_micro <= 0) return hipSuccess;
  const int64_t padded = n_micro + 64;
  uint32_t* keys_a = reinterpret_cast<uint32_t*>(ws);
  uint32_t* keys_b = keys_a + padded;
  uint32_t* idx_a = keys_b + padded;
  uint32_t* idx_b = idx_a + padded;
  int32_t* block_hist = reinterpret_cast<int32_t*>(idx_b + padded);
  const int n_blocks = (int)((n_micro + kSortChunk - 1) / kSortChunk);
  hipLaunchKernelGGL(sort_init_kernel, dim3((unsigned)((n_micro + kSortThreads - 1) / kSortThreads)),
                     dim3(kSortThreads), 0, stream, energy, n_micro, keys_a, idx_a);
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = pass * 8;
    hipLaunchKernelGGL(sort_count_kernel, dim3((unsigned)n_blocks), dim3(kSortThreads), 0, stream, keys_a, n_micro,
                       shift, block_hist);
    hipLaunchKernelGGL(sort_scan_kernel, dim3(1), dim3(kDigits), 0, stream, block_hist, n_blocks);
    hipLaunchKernelGGL(sort_scatter_kernel, dim3((unsigned)n_blocks), dim3(kSortThreads), 0, stream, keys_a, idx_a,
                       n_micro, shift, block_hist, keys_b, idx_b, pass == 3 ? rank : nullptr);
    uint32_t* t = keys_a; keys_a = keys_b; keys_b = t;
    t = idx_a; idx_a = idx_b; idx_b = t;
  }
  return hipGetLastError();
}

}  // namespace camera
