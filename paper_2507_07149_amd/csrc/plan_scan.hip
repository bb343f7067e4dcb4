// Device exclusive prefix scan of per-group packed word counts.
//
// The packed buffer concatenates the groups' codes (paper Sec. 3.3 speaks of packing the
// compressed values together); with a bit width per group the position of group g is the
// sum of the word counts of all groups before it.  Up to kAheadMost groups one launch does it (k_plan_ahead); new widths for a
// plan that exists take one launch as well, from kAheadMostUpdated groups on one whose workgroups tell each other their sums
// (k_plan_once).  A new plan of up to kMaxSummedBlocks blocks of 2048 groups: per-block sums and a second launch in which every
// block adds up the sums before its own and writes its offsets; beyond that a single-block scan of the sums comes between them.
#include "daf_device.h"
#include "daf_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;                          // consecutive groups per thread
constexpr int kBlockGroups = kThreads * kItems;    // 2048

__device__ __forceinline__ uint32_t group_words(uint32_t b, int64_t g, int64_t num_groups, int64_t n,
                                                int32_t gs, int* bad) {
  const bool ok = (b == 1u) | (b == 2u) | (b == 4u) | (b == 8u);
  if (!ok) { *bad = 1; return 0u; }
  const int64_t len = (g == num_groups - 1) ? (n - g * (int64_t)gs) : (int64_t)gs;
  return (uint32_t)((len * b + 31) >> 5);
}

// A thread's kItems consecutive widths: one 8-byte load when all of them exist and the array
// is 8-byte aligned (a thread's first index is a multiple of eight), else byte by byte; entries
// at or past num_groups read as 0.
__device__ __forceinline__ void load_widths(const uint8_t* __restrict__ bits, int64_t base, int64_t num_groups,
                                            uint32_t (&b)[kItems]) {
  static_assert(kItems == 8, "one 8-byte load");
  if (base + kItems <= num_groups && (reinterpret_cast<uintptr_t>(bits) & 7u) == 0u) {
    const uint2 v = *reinterpret_cast<const uint2*>(bits + base);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      b[i] = (v.x >> (8 * i)) & 0xFFu;
      b[4 + i] = (v.y >> (8 * i)) & 0xFFu;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) b[i] = (base + i < num_groups) ? (uint32_t)bits[base + i] : 0u;
  }
}

__device__ __forceinline__ void store_widths(uint8_t* __restrict__ plan_bits, int64_t base, int64_t num_groups,
                                             const uint32_t (&b)[kItems]) {
  if (base + kItems <= num_groups && (reinterpret_cast<uintptr_t>(plan_bits) & 7u) == 0u) {
    uint2 v;
    v.x = b[0] | (b[1] << 8) | (b[2] << 16) | (b[3] << 24);
    v.y = b[4] | (b[5] << 8) | (b[6] << 16) | (b[7] << 24);
    *reinterpret_cast<uint2*>(plan_bits + base) = v;
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (base + i < num_groups) plan_bits[base + i] = (uint8_t)b[i];
  }
}

// Sum over a block, in every thread.
__device__ __forceinline__ unsigned long long block_sum(unsigned long long v, unsigned long long* lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds[wave] = v;
  __syncthreads();
  return lds[0] + lds[1] + lds[2] + lds[3];
}

// Widths outside {1,2,4,8} are replaced by 8 in the plan's copy (so that every kernel that reads
// the copy stays inside its buffers whatever the caller passed) and reported: bit 63 of the
// block's sum carries "this block saw an invalid width".
constexpr unsigned long long kBadBit = 1ull << 63;

__global__ __launch_bounds__(kThreads) void k_plan_block_sums(const uint8_t* __restrict__ src_bits,
                                                              uint8_t* __restrict__ plan_bits,
                                                              int64_t num_groups, int64_t n, int32_t gs,
                                                              unsigned long long* __restrict__ block_sums,
                                                              unsigned long long* __restrict__ posts) {
  if (posts != nullptr && threadIdx.x == 0) {            // a new plan's: empty, and before its first launch of k_plan_once
    posts[blockIdx.x] = 0ull;
    if (blockIdx.x == 0) posts[gridDim.x] = 0ull;
  }
  __shared__ unsigned long long lds[4];
  const int64_t base = (int64_t)blockIdx.x * kBlockGroups + (int64_t)threadIdx.x * kItems;
  unsigned long long s = 0;
  int bad = 0;
  uint32_t b[kItems];
  load_widths(src_bits, base, num_groups, b);
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t g = base + i;
    if (g < num_groups) {
      int bad_here = 0;
      (void)group_words(b[i], g, num_groups, n, gs, &bad_here);
      if (bad_here) { b[i] = 8u; bad = 1; }
      s += group_words(b[i], g, num_groups, n, gs, &bad_here);
    }
  }
  store_widths(plan_bits, base, num_groups, b);
  const int any_bad = __syncthreads_or(bad);
  const unsigned long long tot = block_sum(s, lds);      // far below 2^63
  if (threadIdx.x == 0) block_sums[blockIdx.x] = tot | (any_bad ? kBadBit : 0ull);
}

// One block turns block_sums[] into exclusive offsets in place and writes the grand total: a
// thread sums a run of consecutive entries, the 256 run sums are scanned once, the run is
// rewritten.
__global__ __launch_bounds__(kThreads) void k_plan_scan_block_sums(unsigned long long* __restrict__ block_sums,
                                                                   int64_t n_blocks,
                                                                   unsigned long long* __restrict__ total,
                                                                   int* __restrict__ bad_flag) {
  __shared__ unsigned long long lds[kThreads];
  const int64_t per = (n_blocks + kThreads - 1) / kThreads;
  const int64_t lo = (int64_t)threadIdx.x * per;
  const int64_t hi = lo + per < n_blocks ? lo + per : n_blocks;
  unsigned long long sum = 0;
  int bad = 0;
  for (int64_t i = lo; i < hi; ++i) {
    const unsigned long long v = block_sums[i];
    bad |= (v & kBadBit) ? 1 : 0;
    block_sums[i] = v & ~kBadBit;
    sum += v & ~kBadBit;
  }
  const int any_bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) *bad_flag = any_bad;
  lds[threadIdx.x] = sum;
  __syncthreads();
  unsigned long long acc = sum;                          // Hillis-Steele inclusive scan over the 256 run sums
  for (int o = 1; o < kThreads; o <<= 1) {
    const unsigned long long add = (threadIdx.x >= (unsigned)o) ? lds[threadIdx.x - o] : 0ull;
    __syncthreads();
    acc += add;
    lds[threadIdx.x] = acc;
    __syncthreads();
  }
  unsigned long long run = acc - sum;
  for (int64_t i = lo; i < hi; ++i) {
    const unsigned long long v = block_sums[i];
    block_sums[i] = run;
    run += v;
  }
  if (threadIdx.x == kThreads - 1) *total = acc;
}

// A thread's kItems consecutive offsets from `run` on; whole runs leave in 16-byte stores.
__device__ __forceinline__ void store_offsets(uint32_t* __restrict__ off, int64_t base, int64_t num_groups, uint32_t run,
                                              const uint32_t (&w)[kItems]) {
  uint32_t o[kItems];
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    o[i] = run;
    run += w[i];
  }
  if (base + kItems <= num_groups) {
    *reinterpret_cast<uint4*>(off + base) = make_uint4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<uint4*>(off + base + 4) = make_uint4(o[4], o[5], o[6], o[7]);
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i)
      if (base + i < num_groups) off[base + i] = o[i];
  }
}

// Offsets are kept modulo 2^32 (a plan whose total reaches 2^32 words is rejected from the 64-bit
// total, and its offsets are never used), so the scan inside a block runs on 32-bit values: a
// DPP scan inside each wave, the wave totals through LDS.
// SCANNED: block_sums holds running sums (k_plan_scan_block_sums, which also wrote the total).  Otherwise
// every block adds up the sums before its own, and the last one writes the total and the flag.
template <bool SCANNED>
__global__ __launch_bounds__(kThreads) void k_plan_write_offsets(const uint8_t* __restrict__ bits,
                                                                 int64_t num_groups, int64_t n, int32_t gs,
                                                                 const unsigned long long* __restrict__ block_sums,
                                                                 uint32_t* __restrict__ off,
                                                                 unsigned long long* __restrict__ total,
                                                                 int* __restrict__ bad_flag) {
  __shared__ uint32_t wave_tot[kThreads / daf::kWave];
  __shared__ unsigned long long lds[4];
  const int64_t base = (int64_t)blockIdx.x * kBlockGroups + (int64_t)threadIdx.x * kItems;
  uint32_t b[kItems], w[kItems];
  load_widths(bits, base, num_groups, b);
  uint32_t block_off;
  if (SCANNED) {
    block_off = (uint32_t)block_sums[blockIdx.x];
  } else {
    unsigned long long sum = 0;
    int bad = 0;
    for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kThreads) {
      const unsigned long long v = block_sums[i];
      bad |= (v & kBadBit) ? 1 : 0;
      sum += v & ~kBadBit;
    }
    sum = block_sum(sum, lds);
    block_off = (uint32_t)sum;
    if (blockIdx.x == gridDim.x - 1) {
      const int any_bad = __syncthreads_or(bad);
      const unsigned long long own = block_sums[blockIdx.x];
      if (threadIdx.x == 0) {
        *total = sum + (own & ~kBadBit);
        *bad_flag = (any_bad || (own & kBadBit)) ? 1 : 0;
      }
    }
  }
  uint32_t s = 0;
  int bad_width = 0;
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t g = base + i;
    w[i] = (g < num_groups) ? group_words(b[i], g, num_groups, n, gs, &bad_width) : 0u;
    s += w[i];
  }
  const int lane = threadIdx.x & (daf::kWave - 1), wave = threadIdx.x >> 6;
  const uint32_t incl = daf::wave_inclusive_sum(s);
  if (lane == daf::kWave - 1) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t before = 0u;
#pragma unroll
  for (int v = 0; v < kThreads / daf::kWave; ++v) before += (v < wave) ? wave_tot[v] : 0u;
  store_offsets(off, base, num_groups, block_off + before + incl - s, w);   // the thread's first group
}

// One launch: a workgroup has kItems consecutive groups per thread and adds up the widths of all groups before its own
// for itself.  All those groups are whole ones, so their words are (group size / 32) times the sum of their widths, which
// are sixteen to a load; a few tens of kilobytes from the cache cost less than a second launch.  Reads what other workgroups
// have the copy of: the caller's widths are not the plan's own.
// AHEAD: there are groups before a workgroup's.  Up to kAheadGroups there are none, and the one workgroup goes without the
// loop, its 32 registers of loads and the second sum over the wave.  Launches one behind the other in a graph, 512 / 4096 /
// 8192 groups: with them 4.24 / 4.56 / 5.55 us, without 4.00 / 4.28 / 5.31.
constexpr int kAheadThreads = 1024;
constexpr int kAheadGroups = kItems * kAheadThreads;

// Not 0 where one of the four bytes is none of 1, 2, 4, 8: a bit above the lowest four; more than one bit; no bit (without
// the first no carry leaves a byte).
__device__ __forceinline__ uint32_t wrong_widths(uint32_t w) {
  return (w & 0xF0F0F0F0u) | (w & (w - 0x01010101u)) | (~(w + 0x7F7F7F7Fu) & 0x80808080u);
}
// The four bytes with 8 in the place of every wrong width.
__device__ __forceinline__ uint32_t mended_widths(uint32_t w) {
  for (int j = 0; j < 32; j += 8) {
    const uint32_t b = (w >> j) & 0xFFu;
    if (b != 1u && b != 2u && b != 4u) w = (w & ~(0xFFu << j)) | (8u << j);
  }
  return w;
}

// The sum of the widths of sixteen groups, one to a byte; a width outside {1,2,4,8} counts as 8 and is reported.
__device__ __forceinline__ uint32_t sixteen_widths(const uint4& v, int* bad) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
  uint32_t wrong = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) wrong |= wrong_widths(w[i]);
  if (wrong != 0u) {
    *bad = 1;
    for (int i = 0; i < 4; ++i) w[i] = mended_widths(w[i]);
  }
  uint32_t sum = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_udot4(w[i], 0x01010101u, sum, false);
  return sum;
}

// NEW_PLAN: with posts to empty, as in k_plan_block_sums.  They lie behind the total and the flag: with arguments for them an update of
// 12288 groups took 0.08 us more.
template <bool AHEAD, bool NEW_PLAN>
__global__ __launch_bounds__(kAheadThreads) void k_plan_ahead(const uint8_t* __restrict__ src_bits,
                                                              uint8_t* __restrict__ plan_bits, int64_t num_groups, int64_t n,
                                                              int32_t gs, uint32_t* __restrict__ off,
                                                              unsigned long long* __restrict__ total,
                                                              int* __restrict__ bad_flag) {
  constexpr int kWaves = kAheadThreads / daf::kWave;
  if (NEW_PLAN && blockIdx.x == 0 && threadIdx.x < (num_groups + kBlockGroups - 1) / kBlockGroups + 1) total[2 + threadIdx.x] = 0ull;
  __shared__ uint32_t wave_tot[kWaves];
  [[maybe_unused]] __shared__ uint32_t wave_widths[kWaves];
  __shared__ unsigned long long wave_sum[kWaves];
  const int64_t base = (AHEAD ? (int64_t)blockIdx.x * kAheadGroups : 0) + (int64_t)threadIdx.x * kItems;
  uint32_t w[kItems];
  uint32_t s = 0, widths = 0;
  unsigned long long sum = 0;
  int bad = 0;
  uint32_t b[kItems];
  load_widths(src_bits, base, num_groups, b);
  // the groups before this workgroup's: a multiple of 16
  [[maybe_unused]] const uint4* before_bits = reinterpret_cast<const uint4*>(src_bits);
  const int before_pieces = AHEAD ? (int)(blockIdx.x * (kAheadGroups / 16)) : 0;
  constexpr int kLoads = 8;
  for (int i0 = (int)threadIdx.x; i0 < before_pieces; i0 += kLoads * kAheadThreads) {
    uint4 v[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int i = i0 + j * kAheadThreads;
      v[j] = make_uint4(0x01010101u, 0x01010101u, 0x01010101u, 0x01010101u);
      if (i < before_pieces) v[j] = before_bits[i];
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const uint32_t sixteen = sixteen_widths(v[j], &bad);
      if (i0 + j * kAheadThreads < before_pieces) widths += sixteen;
    }
  }
#pragma unroll
  for (int i = 0; i < kItems; ++i) {
    const int64_t g = base + i;
    w[i] = 0u;
    if (g < num_groups) {
      int bad_here = 0;
      (void)group_words(b[i], g, num_groups, n, gs, &bad_here);
      if (bad_here) { b[i] = 8u; bad = 1; }
      w[i] = group_words(b[i], g, num_groups, n, gs, &bad_here);
    }
    s += w[i];
    sum += w[i];
  }
  store_widths(plan_bits, base, num_groups, b);
  const int lane = threadIdx.x & (daf::kWave - 1), wave = threadIdx.x >> 6;
  const uint32_t incl = daf::wave_inclusive_sum(s), all_widths = AHEAD ? daf::wave_inclusive_sum(widths) : 0u;
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == daf::kWave - 1) {
    wave_tot[wave] = incl;
    if (AHEAD) wave_widths[wave] = all_widths;
    wave_sum[wave] = sum;
  }
  const int any_bad = __syncthreads_or(bad);
  uint32_t before = 0u;
  unsigned long long ahead = 0, own = 0;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    before += (v < wave) ? wave_tot[v] : 0u;
    if (AHEAD) ahead += wave_widths[v];
    own += wave_sum[v];
  }
  if (AHEAD) ahead *= (unsigned long long)((uint32_t)gs / 32u);
  store_offsets(off, base, num_groups, (uint32_t)ahead + before + incl - s, w);
  if (threadIdx.x == 0 && (!AHEAD || blockIdx.x == gridDim.x - 1)) {
    *total = ahead + own;
    *bad_flag = any_bad;                               // of all groups: the last workgroup has read them all
  }
}

// A new plan of up to 65536 groups: k_plan_ahead alone 4.0 ... 5.3 us up to 8192 groups, 5.8 at 10000, 6.4 at 16384, 7.3 at 32768 and 7.4 at
// 65536, the two launches 8.4 from there to 197000; at 197000 groups the sums over all that comes before make it slower (call of
// four launches 62.0 -> 65.4 us, at 524288 51.4 -> 60.3).  An update leaves it for k_plan_once earlier, which a new plan, whose posts are
// not empty yet, cannot take: ahead / once, launches one behind the other: 10000 groups 5.8 / 6.3 us, 12288 5.9 / 6.4, 14336 5.9 / 5.7,
// 16384 6.4 / 5.7, 20480 6.4 / 6.2, 32768 7.3 / 5.9, 65536 7.4 / 5.8.
constexpr int64_t kAheadMost = 1 << 16, kAheadMostUpdated = 7 << 11;
static_assert(kAheadMost / kBlockGroups + 1 <= kAheadThreads, "k_plan_ahead's first workgroup empties the posts");
constexpr int64_t kMaxSummedBlocks = 4096;            // 32 KB of block sums, read by every block
// Rounds of k_plan_once: launches one behind the other, one / two / four rounds, and the form with a launch for the sums (above
// kMaxSummedBlocks two) in front: 70 K groups 6.7 / 8.0 / 10.7, 8.4 us, 197 K 6.6 / 8.2 / 12.0, 8.6, 1 M 7.7 / 8.3 / 11.6, 9.8, 2 M 11.5 /
// 9.3 / 12.0, 12.2, 3 M 15.6 / 11.5 / 12.2, 15.0, 5.6 M 31 / 17 / 14, 23, 9.4 M 76 / 35 / 24, 39, 20 M 176 / 94 / 51, 79, 100 M 1062 / 592 / 314,
// 374, 400 M 4868 / 2270 / 1266, 1606.  (A workgroup of 16384 groups reads 8 bytes for each one before it: at 400 M groups, the most a plan
// has room for being 537 M, 0.1 MB on average, out of the caches.)
constexpr int64_t kOnceRounds2 = 5 << 18, kOnceRounds4 = 13 << 18;

// One launch for any number of groups.  Every workgroup posts the sum of its own groups' words, takes the sums of those before
// it from their posts, all at a time, and writes its offsets: widths are read once, and the second launch, its gap and its reading of
// the widths fall away.  Two launches are bound by latency where there are few groups (197 K: 4.7 + 4.7 us and the gap) and by the rate at
// which waves can be started where there are many (5.6 M in blocks of 2048: 11 + 14.5 us, where 34 MB move): so a thread has
// ROUNDS times kItems groups, every kItems of them behind another's of the same round.
//
// Nothing waits for long: a post that is not there after `polls` looks (about a microsecond each) is done without, and the workgroup adds up
// the widths of all groups before its own itself.  So the result needs no order of the workgroups and no
// two of them at the same time.
//
// Posts stay where they are, and each carries the number of its launch on this plan: rounds.epoch, which every workgroup reads
// before it counts itself in rounds.started, a counter that wraps at the number of workgroups and then moves the epoch on.  A
// workgroup counts itself after its reading, so no launch's number is read again once all launches begun so far are through: whatever
// overlapping updates of one plan leave behind, a later one takes for absent.  (Posts that the last workgroup to finish emptied were
// damaged for good by an overlap.)  Where epochs differ inside overlapping launches, posts are absent and sums worked out.
//
// A post: bits 0 .. 31 the sum, 32 .. 62 the epoch plus one, 63 an invalid width.  Sums of a workgroup's words stay below 2^32:
// group sizes up to kOnceMostSize.
struct OnceRounds {                                      // 0 in a new plan
  uint32_t started, epoch;
};
static_assert(sizeof(OnceRounds) == sizeof(unsigned long long), "one word behind the posts");
constexpr uint32_t kTagMask = 0x7FFFFFFFu;
constexpr int kOnceThreads = 512;
constexpr int32_t kOnceMostSize = 1 << 18;

template <int ROUNDS>
__global__ __launch_bounds__(kOnceThreads) void k_plan_once(const uint8_t* __restrict__ src_bits, uint8_t* __restrict__ plan_bits,
                                                            int64_t num_groups, int64_t n, int32_t gs, uint32_t* __restrict__ off,
                                                            unsigned long long* __restrict__ posts, OnceRounds* __restrict__ launches,
                                                            unsigned long long* __restrict__ total, int* __restrict__ bad_flag,
                                                            int polls) {
  constexpr int kWaves = kOnceThreads / daf::kWave, kRound = kOnceThreads * kItems;
  static_assert((long long)ROUNDS * kRound * (kOnceMostSize / 4) < 1ll << 32, "a workgroup's words in 32 bits");
  __shared__ uint32_t wave_tot[ROUNDS * kWaves];
  __shared__ unsigned long long wave_sum[kWaves];
  __shared__ uint32_t shared_tag;
  // (A cached load, next to the widths: where launches overlap it may be an epoch behind, which is as good as an earlier start.)
  if (threadIdx.x == 0)
    shared_tag = (__hip_atomic_load(&launches->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + 1u) & kTagMask;
  const int64_t first = (int64_t)blockIdx.x * (ROUNDS * kRound);
  const int lane = threadIdx.x & (daf::kWave - 1), wave = threadIdx.x >> 6;
  const uint32_t per_bit = (uint32_t)gs >> 5;            // words of a whole group and bit of width, at most 2^13
  // Eight widths to a register pair.  Where all eight groups are there and none is the tensor's last, sums are dot products and
  // offsets one multiplication each: group by group, 32 groups a thread took 8 us of vector instructions.
  const bool aligned = (reinterpret_cast<uintptr_t>(src_bits) & 7u) == 0u, aligned_copy = (reinterpret_cast<uintptr_t>(plan_bits) & 7u) == 0u;
  auto base_of = [&](int r) { return first + r * kRound + (int64_t)threadIdx.x * kItems; };
  auto whole = [&](int r) { return base_of(r) + kItems < num_groups; };
  auto byte_of = [](const uint2& v, int i) { return ((i < 4 ? v.x : v.y) >> (8 * (i & 3))) & 0xFFu; };
  auto words_of = [&](uint32_t width, int64_t g) {       // of a valid width
    int unused = 0;
    return g == num_groups - 1 ? group_words(width, g, num_groups, n, gs, &unused) : per_bit * width;
  };
  uint2 b[ROUNDS];
  uint32_t s[ROUNDS], incl[ROUNDS];
  int bad = 0;
  if (aligned && first + ROUNDS * kRound < num_groups) {                    // all loads under way together
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) b[r] = *reinterpret_cast<const uint2*>(src_bits + base_of(r));
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      b[r] = make_uint2(0u, 0u);
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        const uint32_t v = base_of(r) + i < num_groups ? (uint32_t)src_bits[base_of(r) + i] : 0u;
        (i < 4 ? b[r].x : b[r].y) |= v << (8 * (i & 3));
      }
    }
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (whole(r)) {
      if ((wrong_widths(b[r].x) | wrong_widths(b[r].y)) != 0u) {
        bad = 1;
        b[r] = make_uint2(mended_widths(b[r].x), mended_widths(b[r].y));
      }
      s[r] = per_bit * __builtin_amdgcn_udot4(b[r].x, 0x01010101u, __builtin_amdgcn_udot4(b[r].y, 0x01010101u, 0u, false), false);
    } else {
      const uint2 mended = make_uint2(mended_widths(b[r].x), mended_widths(b[r].y));
      s[r] = 0u;
      for (int i = 0; i < kItems; ++i) {
        if (base_of(r) + i >= num_groups) break;
        bad |= byte_of(b[r], i) != byte_of(mended, i) ? 1 : 0;
        s[r] += words_of(byte_of(mended, i), base_of(r) + i);
      }
      b[r] = mended;
    }
    incl[r] = daf::wave_inclusive_sum(s[r]);
    if (lane == daf::kWave - 1) wave_tot[r * kWaves + wave] = incl[r];
  }
  const int any_bad = __syncthreads_or(bad);
  uint32_t own = 0u, before[ROUNDS];                     // words of the workgroup, and before the wave's of each round
#pragma unroll
  for (int i = 0; i < ROUNDS * kWaves; ++i) {
    if (i % kWaves == wave) before[i / kWaves] = own;
    own += wave_tot[i];
  }
  const uint32_t tag = shared_tag;
  if (threadIdx.x == 0) {
    __hip_atomic_store(&posts[blockIdx.x], own | (unsigned long long)tag << 32 | (any_bad ? kBadBit : 0ull), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    if (atomicInc(&launches->started, gridDim.x - 1u) == gridDim.x - 1u)
      __hip_atomic_fetch_add(&launches->epoch, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    if (aligned_copy && whole(r)) {
      *reinterpret_cast<uint2*>(plan_bits + base_of(r)) = b[r];
    } else {
      for (int i = 0; i < kItems; ++i)
        if (base_of(r) + i < num_groups) plan_bits[base_of(r) + i] = (uint8_t)byte_of(b[r], i);
    }
  }

  unsigned long long ahead = 0;
  int missed = 0, bad_ahead = 0;
  for (unsigned i = threadIdx.x; i < blockIdx.x; i += kOnceThreads) {
    unsigned long long v = 0;
    bool there = false;
    for (int p = 0; p < polls && !there; ++p) {
      v = __hip_atomic_load(&posts[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      there = ((uint32_t)(v >> 32) & kTagMask) == tag;
    }
    missed |= there ? 0 : 1;
    bad_ahead |= there && (v & kBadBit) ? 1 : 0;
    ahead += (uint32_t)v;
  }
  if (__syncthreads_or(missed)) {
    ahead = 0;
    for (int64_t g0 = (int64_t)threadIdx.x * kItems; g0 < first; g0 += kRound) {
      uint32_t earlier[kItems];
      load_widths(src_bits, g0, num_groups, earlier);
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        int bad_here = 0;
        const uint32_t words = group_words(earlier[i], g0 + i, num_groups, n, gs, &bad_here);
        ahead += bad_here ? 8u * per_bit : words;
        bad_ahead |= bad_here;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) ahead += __shfl_xor(ahead, o);
  if (lane == daf::kWave - 1) wave_sum[wave] = ahead;
  const int any_bad_ahead = __syncthreads_or(bad_ahead);
  ahead = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) ahead += wave_sum[i];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    uint32_t w[kItems];
    if (whole(r)) {
#pragma unroll
      for (int i = 0; i < kItems; ++i) w[i] = __umul24(byte_of(b[r], i), per_bit);
    } else {
#pragma unroll
      for (int i = 0; i < kItems; ++i) w[i] = base_of(r) + i < num_groups ? words_of(byte_of(b[r], i), base_of(r) + i) : 0u;
    }
    store_offsets(off, base_of(r), num_groups, (uint32_t)ahead + before[r] + incl[r] - s[r], w);
  }
  if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) {
    *total = ahead + own;
    *bad_flag = (any_bad || any_bad_ahead) ? 1 : 0;
  }
}

}  // namespace

int64_t daf_plan_scan_blocks(int64_t num_groups) { return (num_groups + kBlockGroups - 1) / kBlockGroups; }

int64_t daf_plan_scan_posts(int64_t num_groups) { return daf_plan_scan_blocks(num_groups) + 1; }

hipError_t daf_launch_plan_scan(const uint8_t* src_bits, uint8_t* plan_bits, int64_t num_groups, int64_t n,
                                int32_t group_size, uint32_t* d_off, unsigned long long* d_block_sums, int64_t n_blocks,
                                unsigned long long* d_total, int* d_bad, unsigned long long* d_posts, bool new_plan,
                                hipStream_t stream, int polls) {
  if (d_posts != d_total + 2) return hipErrorInvalidValue;            // (k_plan_ahead finds them so)
  const bool apart = src_bits + num_groups <= plan_bits || plan_bits + num_groups <= src_bits;
  const bool aligned = (reinterpret_cast<uintptr_t>(src_bits) & 15u) == 0u;
  // (Widths in the plan's own copy would be replaced while others read them.)
  const bool once = !new_plan && num_groups > kAheadMostUpdated && apart && group_size <= kOnceMostSize;
  if (!once && (num_groups <= kAheadGroups || (num_groups <= kAheadMost && apart && aligned))) {
    const unsigned blocks = (unsigned)((num_groups + kAheadGroups - 1) / kAheadGroups);
    const auto kernel = blocks == 1 ? k_plan_ahead<false, false> : new_plan ? k_plan_ahead<true, true> : k_plan_ahead<true, false>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kAheadThreads), 0, stream, src_bits, plan_bits, num_groups, n, group_size, d_off,
                       d_total, d_bad);
    return hipGetLastError();
  }
  if (once) {
    const int rounds = num_groups > kOnceRounds4 ? 4 : num_groups > kOnceRounds2 ? 2 : 1;
    const int64_t per_block = (int64_t)rounds * kOnceThreads * kItems;
    hipLaunchKernelGGL(rounds == 4 ? k_plan_once<4> : rounds == 2 ? k_plan_once<2> : k_plan_once<1>, dim3((unsigned)((num_groups + per_block - 1) / per_block)),
                       dim3(kOnceThreads), 0, stream, src_bits, plan_bits, num_groups, n, group_size, d_off, d_posts,
                       reinterpret_cast<OnceRounds*>(d_posts + n_blocks), d_total, d_bad, polls);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_plan_block_sums, dim3((unsigned)n_blocks), dim3(kThreads), 0, stream, src_bits, plan_bits,
                     num_groups, n, group_size, d_block_sums, new_plan ? d_posts : nullptr);
  if (n_blocks <= kMaxSummedBlocks) {
    hipLaunchKernelGGL(k_plan_write_offsets<false>, dim3((unsigned)n_blocks), dim3(kThreads), 0, stream, plan_bits,
                       num_groups, n, group_size, d_block_sums, d_off, d_total, d_bad);
  } else {
    hipLaunchKernelGGL(k_plan_scan_block_sums, dim3(1), dim3(kThreads), 0, stream, d_block_sums, n_blocks,
                       d_total, d_bad);
    hipLaunchKernelGGL(k_plan_write_offsets<true>, dim3((unsigned)n_blocks), dim3(kThreads), 0, stream, plan_bits,
                       num_groups, n, group_size, d_block_sums, d_off, d_total, d_bad);
  }
  return hipGetLastError();
}
