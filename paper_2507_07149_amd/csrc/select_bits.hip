// Width selection on the device by rank quantiles of the per-group range.
//
// The benchmark workloads assign widths by ranking the groups by (range, group index),
// range = max - min in binary32, and splitting the ranking into C equal parts: rank r gets
// classes[floor(r*C/G)].  This stands in for the paper's controller (Sec. 3.4.1 chooses widths
// from per-activation importance under memory/time budgets); doing it on the device lets the
// sequence statistics -> widths -> plan -> quantize run without the host touching the data.
//
// No sort is needed.  class(g) = number of thresholds k in 1..C-1 with rank(g) >= R_k,
// R_k = ceil(k*G/C).  For each k a radix select (three passes of histograms over the keys, digits
// of 11, 11 and 10 bits, most significant first) finds T_k, the key at sorted position R_k, and
// E_k, how many keys equal to T_k precede that position.  Then rank(g) >= R_k  iff  key_g > T_k,
// or key_g == T_k and g >= I_k, where I_k is the index of the E_k-th (counting from zero) group
// whose key equals T_k.  Keys are the bit patterns of the ranges, which order like the ranges
// because a range is never negative.
//
// Up to kRankMost groups: one launch in which the ranks are counted (k_select_rank); where the widths of an earlier call are
// replaced in place, up to kSmallGroups, one workgroup that keeps the keys in registers (k_select_small).  More, or widths
// over the other inputs: five launches: zero the first counters; write the keys and count their first digit (and zero the
// other counters); count the second digit; count the third; classify, with the keys equal to T_k counted by the way
// (k_select_classify).  What a pass decides (the bin that holds the rank) is worked out from its counters by
// every workgroup of the next launch for itself: a scan of 2048 counters from the cache, next to the
// keys that are on their way, instead of a ticket, a last workgroup and its trips past the caches at the end
// of every launch.  Selection alone, four classes, with tickets and last workgroups in four of six launches, then in six without, now: 500 groups
// 39, 14, 3.9 us (one launch by then), 8192 40, 20, 8.7, 197 K 49, 29, 22.8, 1 M 54, 34, 29, 5.6 M 94, 66, 58; all ranges equal: 197 K 53,
// 38, 25.8, 5.6 M 127, 104, 72.  Six launches and these, random and all equal: 20 M 138 / 121 and 309 / 191, 100 M 640 / 550 and
// 1490 / 942, 400 M 2550 / 2155 and 5980 / 4290.
#include <type_traits>

#include "daf_device.h"
#include "daf_internal.h"

namespace {

using namespace daf;

constexpr int kThreads = 512;
constexpr int kItems = 8;                        // consecutive groups per thread in the ordered passes
constexpr int kBlockGroups = kThreads * kItems;  // 4096
constexpr int kMaxThresholds = 3;                // C <= 4
constexpr int kHistCopies = 2;
constexpr int kBins = 2048;                      // the widest digit has 11 bits
constexpr int kBinsPerThread = kBins / kThreads; // 4
constexpr int kPasses = 3;
constexpr unsigned kMaxWorkgroups = 384;         // of the counting launches, see daf_launch_select_bits
static_assert(kBins % kThreads == 0 && kBinsPerThread == 4, "a thread reads its bins in one 16-byte piece");
constexpr int kLdsCopies0 = 8;                   // copies of a workgroup's own histogram, first pass (one histogram)
constexpr int kLdsCopies = 2;                    // later passes (one histogram per threshold)

__host__ __device__ constexpr int pass_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }
__host__ __device__ constexpr int pass_bits(int pass) { return pass == 2 ? 10 : 11; }

// What is decided after a number of passes, per threshold.
struct Decided {
  uint32_t prefix[kMaxThresholds];      // digits of T_k decided so far
  uint32_t rank[kMaxThresholds];        // rank still to be located inside the prefix bucket; E_k at the end
};
struct SelectState {
  Decided after[kPasses];               // after[p]: passes 0 .. p, written by the launch that follows pass p
  uint32_t pad[2];
  // Counters of the passes, kHistCopies copies, a workgroup adds to copy (its index mod kHistCopies): atomics
  // to one address are served one after the other at the memory side (about 8 ns each), and with few
  // distinct digits every workgroup hits the same few counters.  Few copies, because every workgroup of the next launch
  // reads them all.  (The first pass has one histogram for all thresholds.)
  uint32_t hist[kPasses][kHistCopies][kMaxThresholds][kBins];
};
static_assert(offsetof(SelectState, hist) % 16 == 0, "the counters are read and cleared in 16-byte pieces");

// Zeroes the first pass's counters.
__global__ __launch_bounds__(kThreads) void k_select_init(SelectState* __restrict__ st) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i < kHistCopies * kBins / 4) {
    const int copy = i / (kBins / 4), piece = i % (kBins / 4);
    reinterpret_cast<uint4*>(&st->hist[0][copy][0][0])[piece] = make_uint4(0u, 0u, 0u, 0u);
  }
}

// A workgroup's own histogram in LDS holds COPIES counters per bin, side by side, and a lane adds
// to copy (lane mod COPIES).  The digits of a wave are often few (the leading digit of a range is
// its sign and most of its exponent; ranges of 16-bit tensors have few mantissa bits), and LDS
// atomics of one instruction to one address are served one after the other: the copies divide
// that queue, at no cost in instructions.  (Counting equal digits with ballots first, and adding
// once per distinct digit, took some 40 scalar and vector instructions per call, which was more
// than the queue it avoided.)
template <int COPIES>
__device__ __forceinline__ void hist_add(uint32_t* h, uint32_t digit, bool active) {
  if (active) atomicAdd(&h[digit * COPIES + (threadIdx.x & (COPIES - 1))], 1u);
}
template <int COPIES>
__device__ __forceinline__ uint32_t hist_count(const uint32_t* h, int bin) {
  uint32_t c = 0u;
#pragma unroll
  for (int j = 0; j < COPIES; ++j) c += h[bin * COPIES + j];
  return c;
}

// Exclusive prefix sum of one value per thread over the kThreads threads of a workgroup, and the
// workgroup's total: a DPP scan inside each wave, the wave totals through LDS (two barriers).
__device__ __forceinline__ uint32_t block_exclusive_sum(uint32_t v, uint32_t* wave_tot, uint32_t* total) {
  constexpr int kWaves = kThreads / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_sum(v);
  __syncthreads();                                       // wave_tot may still be read from an earlier call
  if (lane == kWave - 1) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t before = 0u, all = 0u;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t t = wave_tot[w];
    before += (w < wave) ? t : 0u;
    all += t;
  }
  *total = all;
  return before + incl - v;
}

// Thresholds whose prefixes are equal so far select inside the same bucket: they share one
// histogram, that of the first of them.
struct Slices {
  int of[kMaxThresholds];
};
__device__ __forceinline__ Slices shared_slices(const uint32_t (&prefix)[kMaxThresholds], int pass) {
  Slices s;
  s.of[0] = 0;
  s.of[1] = (pass == 0 || prefix[1] == prefix[0]) ? 0 : 1;
  s.of[2] = (pass == 0 || prefix[2] == prefix[0]) ? 0 : (prefix[2] == prefix[1]) ? s.of[1] : 2;
  return s;
}

// The ranks looked for, R_k, before the first pass.
struct Ranks {
  uint32_t r[kMaxThresholds];
};

// The counters of pass PASS that a thread looks at: four consecutive bins of every histogram, all copies added.
template <int PASS>
struct Bins {
  uint4 raw[PASS == 0 ? 1 : kMaxThresholds][kHistCopies];
};
template <int PASS>
__device__ __forceinline__ void load_bins(Bins<PASS>& b, const SelectState* __restrict__ st, int n_thresholds) {
#pragma unroll
  for (int k = 0; k < (PASS == 0 ? 1 : kMaxThresholds); ++k)
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c)
      b.raw[k][c] = k < n_thresholds ? reinterpret_cast<const uint4*>(&st->hist[PASS][c][k][0])[threadIdx.x]
                                     : make_uint4(0u, 0u, 0u, 0u);
}

// Finds for each threshold the bin of pass PASS whose cumulative count first exceeds the rank and extends
// the prefix by that digit; every thread of the workgroup has the result.
template <int PASS>
__device__ __forceinline__ void decide(Decided& d, const Bins<PASS>& bins, int n_thresholds, uint32_t* wave_tot,
                                       Decided* shared) {
  const Slices slices = shared_slices(d.prefix, PASS);
  constexpr int kHists = PASS == 0 ? 1 : kMaxThresholds;
  uint32_t hs[kHists][kBinsPerThread];
#pragma unroll
  for (int k = 0; k < kHists; ++k) {
    uint4 h = bins.raw[k][0];
#pragma unroll
    for (int c = 1; c < kHistCopies; ++c) {
      const uint4 v = bins.raw[k][c];
      h.x += v.x; h.y += v.y; h.z += v.z; h.w += v.w;
    }
    hs[k][0] = h.x; hs[k][1] = h.y; hs[k][2] = h.z; hs[k][3] = h.w;
  }
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    if (k >= n_thresholds) break;
    uint32_t h[kBinsPerThread];
    uint32_t sum = 0u;
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) {
      h[i] = (kHists == 1 || slices.of[k] == 0) ? hs[0][i] : slices.of[k] == 1 ? hs[kHists > 1 ? 1 : 0][i] : hs[kHists > 1 ? 2 : 0][i];
      sum += h[i];
    }
    uint32_t total;
    uint32_t run = block_exclusive_sum(sum, wave_tot, &total);
#pragma unroll
    for (int i = 0; i < kBinsPerThread; ++i) {
      if (run <= d.rank[k] && d.rank[k] < run + h[i]) {       // exactly one bin of one thread (ranks are < G)
        shared->prefix[k] = d.prefix[k] | ((uint32_t)(threadIdx.x * kBinsPerThread + i) << pass_shift(PASS));
        shared->rank[k] = d.rank[k] - run;
      }
      run += h[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    if (k < n_thresholds) {
      d.prefix[k] = shared->prefix[k];
      d.rank[k] = shared->rank[k];
    }
  }
}

// keys[g] = bit pattern of the group's range, and in the same pass the histogram of the keys'
// leading digit (every key counts for every threshold, so one histogram serves all).  A wave
// takes 64 * LOADS consecutive groups per trip, that many loads of each array in flight per lane.
// FROM_SCALE = false: the range is gmax - gmin.  FROM_SCALE = true: gmin holds the groups' scales of
// an earlier quantize call and prev_bits (or, when null, prev_uniform) the widths it ran with; the
// range is scale * (2^b - 1), Eq. 1 (left) turned round, in binary32.
template <bool FROM_SCALE, int LOADS>
__global__ __launch_bounds__(kThreads) void k_select_keys(const float* __restrict__ gmin, const float* __restrict__ gmax,
                                                          const uint8_t* __restrict__ prev_bits, uint32_t prev_uniform,
                                                          int64_t G, uint32_t* __restrict__ keys,
                                                          SelectState* __restrict__ st, int n_thresholds,
                                                          unsigned long long* __restrict__ posts, int64_t n_blocks) {
  constexpr int kLoads = LOADS;
  __shared__ __attribute__((aligned(16))) uint32_t lh[kBins * kLdsCopies0];
  for (int i = threadIdx.x; i < kBins * kLdsCopies0 / 4; i += kThreads)
    reinterpret_cast<uint4*>(lh)[i] = make_uint4(0u, 0u, 0u, 0u);
  {                                                       // the later passes' counters, and the posts
    uint4* later = reinterpret_cast<uint4*>(&st->hist[1][0][0][0]);
    constexpr int kPieces = (kPasses - 1) * kHistCopies * kMaxThresholds * kBins / 4;
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < kPieces; i += gridDim.x * kThreads)
      later[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_blocks; i += (int64_t)gridDim.x * kThreads) posts[i] = 0ull;
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wave_stride = (int64_t)gridDim.x * (kThreads / kWave) * (kWave * kLoads);
  const int64_t first = ((int64_t)blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6)) * (kWave * kLoads);
  for (int64_t g0 = first; g0 < G; g0 += wave_stride) {
    float lo[kLoads], hi[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int64_t g = g0 + j * kWave + lane;
      lo[j] = (g < G) ? gmin[g] : 0.0f;
      if (FROM_SCALE) {
        const uint32_t b = (prev_bits != nullptr && g < G) ? (uint32_t)prev_bits[g] : prev_uniform;
        hi[j] = (float)((1u << (b & 15u)) - 1u);          // L of the earlier call
      } else {
        hi[j] = (g < G) ? gmax[g] : 0.0f;
      }
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int64_t g = g0 + j * kWave + lane;
      const uint32_t key = f2u(FROM_SCALE ? lo[j] * hi[j] : hi[j] - lo[j]);
      if (g < G) keys[g] = key;
      hist_add<kLdsCopies0>(lh, key >> pass_shift(0), g < G);
    }
  }
  __syncthreads();
  if (n_thresholds > 0) {
    for (int i = threadIdx.x; i < kBins; i += kThreads) {
      const uint32_t c = hist_count<kLdsCopies0>(lh, i);
      if (c) atomicAdd(&st->hist[0][blockIdx.x % kHistCopies][0][i], c);
    }
  }
}

// What is decided after pass PASS, from its counters (every thread has the result).
template <int PASS>
__device__ __forceinline__ Decided decided_after(SelectState* __restrict__ st, const Ranks& ranks, int n_thresholds,
                                                 uint32_t* wave_tot, Decided* shared) {
  Bins<PASS> bins;
  load_bins<PASS>(bins, st, n_thresholds);
  Decided d;
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    d.prefix[k] = PASS == 0 ? 0u : st->after[PASS == 0 ? 0 : PASS - 1].prefix[k];
    d.rank[k] = PASS == 0 ? ranks.r[k] : st->after[PASS == 0 ? 0 : PASS - 1].rank[k];
  }
  decide<PASS>(d, bins, n_thresholds, wave_tot, shared);
  if (blockIdx.x == 0 && threadIdx.x == 0) st->after[PASS] = d;      // for the launches after this one
  return d;
}

// Histogram of the PASS-th digit among the keys whose higher digits equal the prefix.
template <int PASS, int LOADS>
__global__ __launch_bounds__(kThreads) void k_select_hist(const uint32_t* __restrict__ keys, int64_t G,
                                                          SelectState* __restrict__ st, Ranks ranks, int n_thresholds) {
  constexpr int kShift = pass_shift(PASS), kDigitBins = 1 << pass_bits(PASS);
  __shared__ __attribute__((aligned(16))) uint32_t lh[kMaxThresholds][kBins * kLdsCopies];
  __shared__ uint32_t wave_tot[kThreads / kWave];
  __shared__ Decided shared;
  for (int i = threadIdx.x; i < kMaxThresholds * kBins * kLdsCopies / 4; i += kThreads)
    reinterpret_cast<uint4*>(&lh[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  const Decided d = decided_after<PASS - 1>(st, ranks, n_thresholds, wave_tot, &shared);
  const uint32_t(&prefix)[kMaxThresholds] = d.prefix;
  const Slices slices = shared_slices(prefix, PASS);
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  // LOADS 16-byte loads per lane and trip issued together (the key array is padded to whole chunks), so that enough bytes are in
  // flight; a wave takes 64 * LOADS consecutive chunks.
  constexpr int kLoads = LOADS;
  const int64_t n_chunks = (G + 3) >> 2;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wave_stride = stride / kWave * (kWave * kLoads);
  const int64_t first = ((int64_t)blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6)) * (kWave * kLoads);
  for (int64_t c0 = first; c0 < n_chunks; c0 += wave_stride) {
    uint4 v[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int64_t c = c0 + j * kWave + lane;
      v[j] = make_uint4(0u, 0u, 0u, 0u);
      if (c < n_chunks) v[j] = reinterpret_cast<const uint4*>(keys)[c];
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int64_t c = c0 + j * kWave + lane;
      const uint32_t key4[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = c * 4 + e < G;
        const uint32_t key = key4[e];
        const uint32_t digit = (key >> kShift) & (uint32_t)(kDigitBins - 1);
#pragma unroll
        for (int k = 0; k < kMaxThresholds; ++k) {
          if (k >= n_thresholds || slices.of[k] != k) continue;   // counted with an earlier threshold
          hist_add<kLdsCopies>(lh[k], digit, in && (((key ^ prefix[k]) >> (kShift + pass_bits(PASS))) == 0u));
        }
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n_thresholds * kBins; i += kThreads) {
    const int k = i / kBins;
    const uint32_t c = hist_count<kLdsCopies>(lh[k], i % kBins);
    const bool own = k == 0 || (k == 1 ? slices.of[1] == 1 : slices.of[2] == 2);
    if (c && own) atomicAdd(&(&st->hist[PASS][blockIdx.x % kHistCopies][0][0])[i], c);
  }
}

// A thread's kItems consecutive keys: two 16-byte loads (the key array is padded to a multiple
// of four entries and 16-byte aligned, and a thread's first index is a multiple of eight);
// entries at or past G read as 0xFFFFFFFF.
__device__ __forceinline__ void load_keys(const uint32_t* __restrict__ keys, int64_t base, int64_t G,
                                          uint32_t (&key)[kItems]) {
  static_assert(kItems == 8, "two uint4 loads");
  const int64_t padded = (G + 3) & ~(int64_t)3;
  uint4 a = make_uint4(~0u, ~0u, ~0u, ~0u), b = a;
  if (base < padded) a = *reinterpret_cast<const uint4*>(keys + base);
  if (base + 4 < padded) b = *reinterpret_cast<const uint4*>(keys + base + 4);
  key[0] = a.x; key[1] = a.y; key[2] = a.z; key[3] = a.w;
  key[4] = b.x; key[5] = b.y; key[6] = b.z; key[7] = b.w;
#pragma unroll
  for (int i = 0; i < kItems; ++i)
    if (base + i >= G) key[i] = 0xFFFFFFFFu;
}

// Eight widths of consecutive groups, bytes of two words, `count` of them inside the array.
__device__ __forceinline__ void store_widths(uint8_t* __restrict__ out, const uint8_t (&w)[kItems], int64_t count) {
  if (count >= kItems && (reinterpret_cast<uintptr_t>(out) & 7u) == 0u) {
    const uint2 v = make_uint2((uint32_t)w[0] | ((uint32_t)w[1] << 8) | ((uint32_t)w[2] << 16) | ((uint32_t)w[3] << 24),
                               (uint32_t)w[4] | ((uint32_t)w[5] << 8) | ((uint32_t)w[6] << 16) | ((uint32_t)w[7] << 24));
    *reinterpret_cast<uint2*>(out) = v;                   // eight widths in one store
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (i < count) out[i] = w[i];
  }
}

// rank(g) >= R_k  iff  key_g > T_k, or key_g == T_k and at least E_k equal keys come before g.  A block of 4096 groups posts
// how many of its keys equal each T_k, and one that has such keys takes the counts of the blocks before it from their posts.
// (Counting in a launch of its own and classifying in the next: 197 K groups 4.4 + 5.2 us and the gap.)
// Nothing waits for long: a post that is not there after `polls` looks (about a microsecond each) is done without, and the block
// counts the equal keys before its own itself.  So the result needs no order of the workgroups and no two of them
// at the same time.  The posts were emptied by k_select_keys.
constexpr unsigned long long kPosted = 1ull << 63;
constexpr int kPostBits = 16;                            // of one threshold's count, at most kBlockGroups
// ROUNDS: a workgroup has that many blocks of 4096 groups, a wave the 512 * ROUNDS next to each other (what is decided
// is worked out once for all of them, and fewer waves have to be started).
constexpr int kMostRounds = 2;
static_assert(kMostRounds * kBlockGroups < 1 << kPostBits && kMaxThresholds * kPostBits < 63, "a post holds the counts of all thresholds");

template <int ROUNDS>
__global__ __launch_bounds__(kThreads) void k_select_classify(const uint32_t* __restrict__ keys, int64_t G,
                                                              SelectState* __restrict__ st, Ranks ranks, int n_thresholds,
                                                              uint32_t classes_packed, unsigned long long* __restrict__ posts,
                                                              int polls, uint8_t* __restrict__ out_bits) {
  constexpr int kWaves = kThreads / kWave, kWaveGroups = kWave * kItems;
  __shared__ uint32_t wave_tot[kWaves], wave_equal[kMaxThresholds][kWaves], wave_ahead[kMaxThresholds][kWaves];
  __shared__ Decided shared;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  const int64_t first = (int64_t)blockIdx.x * (ROUNDS * kBlockGroups);
  auto base_of = [&](int r) { return first + (wave * ROUNDS + r) * kWaveGroups + lane * kItems; };
  uint32_t key[ROUNDS][kItems], cls[ROUNDS][kItems];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    load_keys(keys, base_of(r), G, key[r]);
#pragma unroll
    for (int i = 0; i < kItems; ++i) cls[r][i] = 0u;
  }
  if (n_thresholds > 0) {
    const Decided d = decided_after<kPasses - 1>(st, ranks, n_thresholds, wave_tot, &shared);
    uint32_t before[kMaxThresholds][ROUNDS];             // equal keys before a thread's first of a round, in the wave, then in all
#pragma unroll
    for (int k = 0; k < kMaxThresholds; ++k) {
      uint32_t carry = 0u;
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
        before[k][r] = 0u;
        if (k >= n_thresholds || d.rank[k] == 0u) continue;            // (E_k = 0: every equal key counts)
        uint32_t mine = 0u;
#pragma unroll
        for (int i = 0; i < kItems; ++i) mine += (base_of(r) + i < G && key[r][i] == d.prefix[k]) ? 1u : 0u;
        const uint32_t incl = wave_inclusive_sum(mine);
        before[k][r] = carry + incl - mine;
        carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
      }
      if (lane == 0) wave_equal[k][wave] = carry;
    }
    __syncthreads();
    uint32_t wanted = 0u;
    unsigned long long post = kPosted;
#pragma unroll
    for (int k = 0; k < kMaxThresholds; ++k) {
      uint32_t earlier = 0u, total = 0u;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        const uint32_t c = wave_equal[k][v];
        earlier += v < wave ? c : 0u;
        total += c;
      }
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) before[k][r] += earlier;
      post |= (unsigned long long)total << (k * kPostBits);
      wanted |= total;
    }
    if (threadIdx.x == 0) __hip_atomic_store(&posts[blockIdx.x], post, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (wanted != 0u && blockIdx.x > 0u) {               // (the same in all threads)
      uint32_t c[kMaxThresholds] = {0u, 0u, 0u};
      int missed = 0;
      for (unsigned i = threadIdx.x; i < blockIdx.x; i += kThreads) {
        unsigned long long v = 0ull;
        for (int p = 0; p < polls && !(v & kPosted); ++p) v = __hip_atomic_load(&posts[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        missed |= (v & kPosted) ? 0 : 1;
#pragma unroll
        for (int k = 0; k < kMaxThresholds; ++k) c[k] += (uint32_t)(v >> (k * kPostBits)) & ((1u << kPostBits) - 1u);
      }
      if (__syncthreads_or(missed)) {
#pragma unroll
        for (int k = 0; k < kMaxThresholds; ++k) c[k] = 0u;
        for (int64_t g0 = (int64_t)threadIdx.x * kItems; g0 < first; g0 += kBlockGroups) {
          uint32_t other[kItems];
          load_keys(keys, g0, G, other);
#pragma unroll
          for (int i = 0; i < kItems; ++i)
#pragma unroll
            for (int k = 0; k < kMaxThresholds; ++k) c[k] += k < n_thresholds && other[i] == d.prefix[k] ? 1u : 0u;
        }
      }
#pragma unroll
      for (int k = 0; k < kMaxThresholds; ++k) {
        const uint32_t sum = wave_inclusive_sum(c[k]);
        if (lane == kWave - 1) wave_ahead[k][wave] = sum;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kMaxThresholds; ++k)
#pragma unroll
        for (int v = 0; v < kWaves; ++v)
#pragma unroll
          for (int r = 0; r < ROUNDS; ++r) before[k][r] += wave_ahead[k][v];
    }
#pragma unroll
    for (int k = 0; k < kMaxThresholds; ++k) {
      if (k >= n_thresholds) continue;
      const uint32_t T = d.prefix[k], E = d.rank[k];
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r) {
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
          const bool equal = key[r][i] == T;
          if (key[r][i] > T || (equal && before[k][r] >= E)) ++cls[r][i];
          before[k][r] += equal ? 1u : 0u;
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    uint8_t w[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) w[i] = (uint8_t)(classes_packed >> (8u * cls[r][i]));
    if (base_of(r) < G) store_widths(out_bits + base_of(r), w, G - base_of(r));
  }
}

// ---- few groups: one workgroup, the keys in registers ------------------------------------------------------------
// kItems consecutive groups per thread (so that equal keys are met in group order), 1024 threads; every
// pass counts into LDS, finds the bins and goes on.
constexpr int kSmallThreads = 1024;
constexpr int64_t kSmallGroups = 8 * kSmallThreads;

__device__ __forceinline__ uint32_t small_exclusive_sum(uint32_t v, uint32_t* wave_tot) {
  constexpr int kWaves = kSmallThreads / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_sum(v);
  __syncthreads();
  if (lane == kWave - 1) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t before = 0u;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) before += (w < wave) ? wave_tot[w] : 0u;
  return before + incl - v;
}

template <int PASS>
__device__ __forceinline__ void small_pass(const uint32_t (&key)[kItems], int64_t base, int64_t G, Decided& d, int n_thresholds,
                                           uint32_t* lh, uint32_t* wave_tot, Decided* shared) {
  constexpr int kShift = pass_shift(PASS), kDigitBins = 1 << pass_bits(PASS);
  constexpr int kCopies = PASS == 0 ? kLdsCopies0 : kLdsCopies, kHists = PASS == 0 ? 1 : kMaxThresholds;
  static_assert(kHists * kCopies * kBins <= kLdsCopies0 * kBins, "the first pass takes the most LDS");
  const Slices slices = shared_slices(d.prefix, PASS);
  __syncthreads();                                         // the counters may still be read
  for (int i = threadIdx.x; i < kHists * kCopies * kDigitBins / 4; i += kSmallThreads)
    reinterpret_cast<uint4*>(lh)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const uint32_t digit = (key[i] >> kShift) & (uint32_t)(kDigitBins - 1);
#pragma unroll
    for (int k = 0; k < kHists; ++k) {
      if (k >= n_thresholds || slices.of[k] != k) continue;
      bool in = base + i < G;
      if constexpr (PASS > 0) in = in && (((key[i] ^ d.prefix[k]) >> (kShift + pass_bits(PASS))) == 0u);
      hist_add<kCopies>(lh + k * kCopies * kDigitBins, digit, in);
    }
  }
  __syncthreads();
  constexpr int kPer = kDigitBins / kSmallThreads;         // 2 or 1 bins per thread
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    if (k >= n_thresholds) break;
    const uint32_t* h = lh + slices.of[k] * kCopies * kDigitBins;
    uint32_t c[kPer], sum = 0u;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      c[i] = hist_count<kCopies>(h, threadIdx.x * kPer + i);
      sum += c[i];
    }
    uint32_t run = small_exclusive_sum(sum, wave_tot);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (run <= d.rank[k] && d.rank[k] < run + c[i]) {
        shared->prefix[k] = d.prefix[k] | ((uint32_t)(threadIdx.x * kPer + i) << kShift);
        shared->rank[k] = d.rank[k] - run;
      }
      run += c[i];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    if (k < n_thresholds) {
      d.prefix[k] = shared->prefix[k];
      d.rank[k] = shared->rank[k];
    }
  }
}

// Only with the scales and widths of an earlier call; the new widths may lie over either: all are read before the first
// barrier, and nothing is written before the last.
__global__ __launch_bounds__(kSmallThreads) void k_select_small(const float* scale, const uint8_t* prev_bits, int64_t G,
                                                                Ranks ranks, int n_thresholds, uint32_t classes_packed,
                                                                uint8_t* out_bits) {
  __shared__ __attribute__((aligned(16))) uint32_t lh[kBins * kLdsCopies0];
  __shared__ uint32_t wave_tot[kSmallThreads / kWave];
  __shared__ Decided shared;
  const int64_t base = (int64_t)threadIdx.x * kItems;
  uint32_t key[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t g = base + i;
    key[i] = g < G ? f2u(scale[g] * (float)((1u << (prev_bits[g] & 15u)) - 1u)) : 0xFFFFFFFFu;
  }
  Decided d;
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    d.prefix[k] = 0u;
    d.rank[k] = ranks.r[k];
  }
  if (n_thresholds > 0) {
    small_pass<0>(key, base, G, d, n_thresholds, lh, wave_tot, &shared);
    small_pass<1>(key, base, G, d, n_thresholds, lh, wave_tot, &shared);
    small_pass<2>(key, base, G, d, n_thresholds, lh, wave_tot, &shared);
  }
  uint32_t cls[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) cls[i] = 0u;
#pragma unroll
  for (int k = 0; k < kMaxThresholds; ++k) {
    if (k >= n_thresholds) break;
    const uint32_t T = d.prefix[k], E = d.rank[k];
    uint32_t mine = 0u;
#pragma unroll
    for (int i = 0; i < kItems; ++i) mine += (base + i < G && key[i] == T) ? 1u : 0u;
    uint32_t before = small_exclusive_sum(mine, wave_tot);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const bool equal = key[i] == T;
      if (key[i] > T || (equal && before >= E)) ++cls[i];
      before += equal ? 1u : 0u;
    }
  }
  uint8_t w[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) w[i] = (uint8_t)(classes_packed >> (8u * cls[i]));
  if (base < G) store_widths(out_bits + base, w, G - base);
}

// Few groups, ranks counted outright: a workgroup has kRankGroups groups, all keys in LDS, and counts for each of its
// groups the keys that come before it, (range, index), a thread 1 / kRankParts of them.  No passes, no counters, one barrier
// before the counting and one behind it.  Every workgroup reads all groups, so the widths written are not those read.
constexpr int kRankThreads = 1024;
constexpr int kRankGroups = 32, kRankParts = kRankThreads / kRankGroups;
// Four classes, launches one behind the other, 512 / 2048 / 4096 / 8192 groups: one workgroup with the keys in registers 13.2 / 13.8 /
// 15.0 / 17.6 us, five launches 18.9 / 19.4 / 19.7 / 19.8, this 3.9 / 4.8 / 6.0 / 8.7; 12000: 17 against 20.1 in five.  The work grows with the
// square, and the keys fill the LDS at 16384 groups; there, five / this: random ranges, four / three / two classes 22.3 / 21.7, 20.2 / 20.8,
// 18.1 / 20.8, maxima of a gelu's groups 23.7 / 21.6, 21.1 / 20.8, 19.3 / 20.8, all equal 23.9 / 21.2, 21.9 / 20.8, 19.7 / 20.8; another card, random, four
// classes 20.2 / 21.7.
constexpr int64_t kRankMost = 16 << 10;

template <bool FROM_SCALE>
__global__ __launch_bounds__(kRankThreads) void k_select_rank(const float* __restrict__ gmin, const float* __restrict__ gmax,
                                                              const uint8_t* __restrict__ prev_bits, uint32_t prev_uniform,
                                                              int G, Ranks ranks, int n_thresholds, uint32_t classes_packed,
                                                              uint8_t* __restrict__ out_bits) {
  extern __shared__ __attribute__((aligned(16))) uint32_t keys[];         // G, then kRankParts x kRankGroups counts
  const int padded = (G + 2 * kRankGroups - 1) / (2 * kRankGroups) * (2 * kRankGroups);
  uint32_t* counts = keys + padded;
  const int t = (int)threadIdx.x;
  constexpr int kLoads = 8;
  for (int g0 = t; g0 < padded; g0 += kLoads * kRankThreads) {
    float lo[kLoads], hi[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int g = g0 + j * kRankThreads;
      lo[j] = g < G ? gmin[g] : 0.0f;
      if (FROM_SCALE) {
        const uint32_t b = (prev_bits != nullptr && g < G) ? (uint32_t)prev_bits[g] : prev_uniform;
        hi[j] = (float)((1u << (b & 15u)) - 1u);
      } else {
        hi[j] = g < G ? gmax[g] : 0.0f;
      }
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int g = g0 + j * kRankThreads;
      // (behind the last group the highest key: nothing comes after it, and groups of that key have lower indexes)
      if (g < padded) keys[g] = g < G ? f2u(FROM_SCALE ? lo[j] * hi[j] : hi[j] - lo[j]) : 0xFFFFFFFFu;
    }
  }
  __syncthreads();

  // Part p counts in the blocks of 32 keys p, p + kRankParts, ...: the two halves of a wave in neighbouring blocks.
  const int tile = (int)blockIdx.x, me = t & (kRankGroups - 1), part = t / kRankGroups;
  const int i = tile * kRankGroups + me;
  const uint32_t key = keys[i];                                            // (i < padded)
  const int blocks = padded / kRankGroups;                                 // even
  uint32_t before = 0u;
  for (int block = part; block < blocks; block += kRankParts) {
    const uint4* k4 = reinterpret_cast<const uint4*>(keys + block * kRankGroups);
    const int pair = __builtin_amdgcn_readfirstlane(block) >> 1;           // of the wave's two blocks
    if (pair < tile >> 1) {                                                // all before i: an equal key comes first
#pragma unroll
      for (int q = 0; q < kRankGroups / 4; ++q) {
        const uint4 v = k4[q];
        before += (v.x <= key) + (v.y <= key) + (v.z <= key) + (v.w <= key);
      }
    } else if (pair > tile >> 1) {
#pragma unroll
      for (int q = 0; q < kRankGroups / 4; ++q) {
        const uint4 v = k4[q];
        before += (v.x < key) + (v.y < key) + (v.z < key) + (v.w < key);
      }
    } else {
#pragma unroll
      for (int q = 0; q < kRankGroups / 4; ++q) {
        const uint4 v = k4[q];
        const uint32_t k[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) before += k[e] < key || (k[e] == key && block * kRankGroups + 4 * q + e < i);
      }
    }
  }
  counts[part * kRankGroups + me] = before;
  __syncthreads();
  if (t < kRankGroups && i < G) {
    uint32_t rank = 0u;
#pragma unroll
    for (int p = 0; p < kRankParts; ++p) rank += counts[p * kRankGroups + t];
    uint32_t cls = 0u;
    for (int k = 0; k < n_thresholds; ++k) cls += rank >= ranks.r[k] ? 1u : 0u;
    out_bits[i] = (uint8_t)(classes_packed >> (8u * cls));
  }
}

// Keys per thread and trip in the launches that write and count them (2 / 4, 8 / 8, 8 / 16: the writing launch, the counting ones).  Few make more
// workgroups, whose start and counting take less time, but each adds its counts to the shared ones.  Selection alone, four classes: 65 K
// groups 21.0 / 22.5 / 24.1 us, 131 K 21.7 / 22.6 / 24.0, 197 K 23.2 / 22.9 / 24.4, 400 K 27.9 / 24.5 / 25.4, 700 K 35.9 / 28.9 / 28.8.
constexpr int64_t kFewKeys = 5 << 15, kManyKeys = 1 << 19;
// Rounds of k_select_classify: selection alone, four classes, launches one behind the other, one / two / four rounds: 197 K groups 24.2 / 25.6 /
// 29.5 us, 1.5 M 35.9 / 37.0 / 41.5, 2 M 39.1 / 37.6 / 44.1, 5.6 M 60.6 / 58.1 / 64.0 (from here on all with 8 and 16 keys to a thread).  Six
// launches before: 27.0, 39.2, 40.6, 62.9.  One / two rounds with all ranges equal, where every workgroup reads all posts before its own: 1.5 M
// 36.3 / 36.3, 5.6 M 77 / 72, 20 M 210 / 196.
constexpr int64_t kClassifyRounds2 = 7 << 18;

}  // namespace

int64_t daf_select_bits_workspace_size(int64_t G) {
  const int64_t n_blocks = (G + kBlockGroups - 1) / kBlockGroups;
  return (int64_t)sizeof(SelectState) + ((G + 3) / 4) * 16 + kMaxThresholds * ((n_blocks + 3) / 4) * 16 + 64;
}

hipError_t daf_launch_select_bits(const float* gmin, const float* gmax, const uint8_t* prev_bits, int32_t prev_uniform,
                                  int64_t G, const uint8_t* classes, int n_classes, uint8_t* out_bits, void* workspace,
                                  hipStream_t stream, int polls) {
  SelectState* st = static_cast<SelectState*>(workspace);
  uint32_t* keys = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + ((sizeof(SelectState) + 15) / 16) * 16);
  unsigned long long* posts = reinterpret_cast<unsigned long long*>(keys + ((G + 3) / 4) * 4);      // a multiple of 16 bytes in
  const int64_t n_blocks = (G + kBlockGroups - 1) / kBlockGroups;

  // thresholds R_k = ceil(k*G/C) that some rank can reach (R_k < G); the rest never apply
  Ranks ranks = {{0u, 0u, 0u}};
  int n_thr = 0;
  for (int k = 1; k < n_classes; ++k) {
    const int64_t r = (k * G + n_classes - 1) / n_classes;
    if (r < G) ranks.r[n_thr++] = (uint32_t)r;
  }
  uint32_t packed = 0;
  for (int c = 0; c < n_classes; ++c) packed |= (uint32_t)classes[c] << (8 * c);
  // thresholds skipped because R_k >= G sit at the end (R_k grows with k), so class = number of
  // satisfied thresholds still indexes `classes` correctly.

  // The widths may replace an input, the earlier widths above all: then nothing may be written before all has been read.
  auto clear_of = [&](const void* input, int64_t bytes) {
    const uint8_t* p = static_cast<const uint8_t*>(input);
    return p == nullptr || out_bits + G <= p || p + bytes <= out_bits;
  };
  const bool apart = clear_of(prev_bits, G) && clear_of(gmin, 4 * G) && clear_of(gmax, 4 * G);
  if (G <= kRankMost && apart) {
    const unsigned blocks = (unsigned)((G + kRankGroups - 1) / kRankGroups);
    const unsigned lds_bytes = (unsigned)(((G + 2 * kRankGroups - 1) / (2 * kRankGroups) * (2 * kRankGroups) + kRankThreads) * 4);
    if (gmax != nullptr)
      hipLaunchKernelGGL(k_select_rank<false>, dim3(blocks), dim3(kRankThreads), lds_bytes, stream, gmin, gmax, nullptr, 0u,
                         (int)G, ranks, n_thr, packed, out_bits);
    else
      hipLaunchKernelGGL(k_select_rank<true>, dim3(blocks), dim3(kRankThreads), lds_bytes, stream, gmin, nullptr, prev_bits,
                         (uint32_t)prev_uniform, (int)G, ranks, n_thr, packed, out_bits);
    return hipGetLastError();
  }
  // The widths replace an input, few groups: one launch of one workgroup, 13.2 us at 512 groups to 17.6 at kSmallGroups, where the five
  // launches take 18.9 to 20.2; with two and four times as many keys per thread it took 32 and 59.
  if (G <= kSmallGroups && prev_bits != nullptr) {
    hipLaunchKernelGGL(k_select_small, dim3(1), dim3(kSmallThreads), 0, stream, gmin, prev_bits, G, ranks, n_thr, packed,
                       out_bits);
    return hipGetLastError();
  }

  // The counting launches take at most kMaxWorkgroups workgroups of 8 waves: each adds its non-zero
  // counts to the shared counters, and those are served one after the other per address (5.6 M groups: 66 us
  // with 256, 384 and 512 workgroups, 73 with 768).
  const unsigned cap = kMaxWorkgroups;
  hipLaunchKernelGGL(k_select_init, dim3((kHistCopies * kBins / 4 + kThreads - 1) / kThreads), dim3(kThreads), 0, stream, st);
  const int key_loads = G > kFewKeys ? 8 : 2, loads = G > kManyKeys ? 4 : G > kFewKeys ? 2 : 1;
  auto workgroups = [&](int64_t per_thread) {
    const int64_t n = (G + per_thread * kThreads - 1) / (per_thread * kThreads);
    return dim3((unsigned)(n < cap ? n : cap));
  };
  const auto write_keys = gmax != nullptr ? (key_loads == 8 ? k_select_keys<false, 8> : k_select_keys<false, 2>)
                                          : (key_loads == 8 ? k_select_keys<true, 8> : k_select_keys<true, 2>);
  hipLaunchKernelGGL(write_keys, workgroups(key_loads), dim3(kThreads), 0, stream, gmin, gmax, gmax != nullptr ? nullptr : prev_bits,
                     gmax != nullptr ? 0u : (uint32_t)prev_uniform, G, keys, st, n_thr, posts, n_blocks);
  if (n_thr > 0) {
    auto count = [&](auto pass) {
      constexpr int P = decltype(pass)::value;
      const auto kernel = loads == 4 ? k_select_hist<P, 4> : loads == 2 ? k_select_hist<P, 2> : k_select_hist<P, 1>;
      hipLaunchKernelGGL(kernel, workgroups(4 * loads), dim3(kThreads), 0, stream, keys, G, st, ranks, n_thr);
    };
    count(std::integral_constant<int, 1>{});
    count(std::integral_constant<int, 2>{});
  }
  const int rounds = G > kClassifyRounds2 ? 2 : 1;
  hipLaunchKernelGGL(rounds == 2 ? k_select_classify<2> : k_select_classify<1>,
                     dim3((unsigned)((n_blocks + rounds - 1) / rounds)), dim3(kThreads), 0, stream, keys, G, st, ranks, n_thr, packed,
                     posts, polls, out_bits);
  return hipGetLastError();
}
