// Route "tile": group sizes that are a power of two up to 4096, one wave per tile.
#pragma once
#include "quantize_common.h"
#include "quantize_group.h"

namespace {

// ------------------------------------------------------------------------------------------
// Fast path: one wave per tile.
// ------------------------------------------------------------------------------------------
// Lane l of load u holds the 16-byte chunk u*64 + l of the tile.  A group spans
// 2^LPG_LOG2 consecutive chunks: up to 64 neighbouring lanes of one load (LPG_LOG2 <= 6), or
// the whole wave over 2, 4, 8 or 16 consecutive loads (LPG_LOG2 = 7..10).
// DIV = 2: a tile of half the size (2048 elements of a 16-bit format): twice as many, shorter
// waves, for tensors so small that whole-size tiles would leave the last round of waves half
// empty.
template <int DT, int LPG_LOG2, int DIV = 1>
struct TileShape {
  static constexpr int kEpl = ElemTraits<DT>::kPerLoad;            // elements per lane per load
  static constexpr int kLaneLog2 = LPG_LOG2 < 6 ? LPG_LOG2 : 6;    // log2 lanes of a group in one load
  static constexpr int kLpg = 1 << kLaneLog2;                      // lanes per group (in one load)
  static constexpr int kGpl = kWave / kLpg;                        // group segments per load
  static constexpr int kLoadsPerGroup = 1 << (LPG_LOG2 - kLaneLog2);
  static constexpr int kMaxLoads = 4096 / (kWave * kEpl) / DIV;    // 16 (fp32) or 8 (16-bit), over DIV
  static constexpr int kLoads = (kMaxLoads * kGpl <= kWave) ? kMaxLoads : kWave / kGpl;
  static constexpr int kSegments = kLoads * kGpl;                  // (load, lane run) pairs, <= 64
  static constexpr int kGroups = kSegments / kLoadsPerGroup;       // groups per tile
  static constexpr int kElems = kLoads * kWave * kEpl;             // 2048 or 4096
  static constexpr int kGroupSize = (1 << LPG_LOG2) * kEpl;
  static constexpr int kPhilox = kElems / kElemsPerPhilox / kWave; // Philox calls per lane
  static constexpr bool kValid = kLoadsPerGroup <= kLoads && kElems >= kElemsPerPhilox * kWave;
  static_assert(kSegments <= kWave, "tile shape");
};

// The tile the quantize kernels use for a group shape.  binary32 tiles are a quarter of the
// largest size (1024 elements, 4 loads per lane; a half where a group needs more loads): the
// binary32 kernel is bound by memory, and with a third of the registers per wave more waves keep
// loads in flight.  Measured, whole / half / quarter tiles: 40.6 / 37.0 / 35.2 us on a
// 51 M-element tensor, 150 / 141 / 131 us on 205 M elements.  The 16-bit kernels are bound by
// vector instructions and lose to the per-tile overhead of smaller tiles (measured), so they keep
// the whole size.
template <int DT, int LPG_LOG2>
constexpr int tile_div() {
  if (DT != kF32) return 1;
  if (TileShape<DT, LPG_LOG2, 4>::kValid && TileShape<DT, LPG_LOG2, 4>::kElems < TileShape<DT, LPG_LOG2, 2>::kElems) return 4;
  if (TileShape<DT, LPG_LOG2, 2>::kValid && TileShape<DT, LPG_LOG2, 2>::kElems < TileShape<DT, LPG_LOG2, 1>::kElems) return 2;
  return 1;
}
template <int DT, int LPG_LOG2>
using QTile = TileShape<DT, LPG_LOG2, tile_div<DT, LPG_LOG2>()>;

struct alignas(16) GroupInfo {   // what every lane of a group needs for the element map
  float mn;
  float invs;                    // inv*256, or inv on the two-multiplication path
  uint32_t b;                    // width; bits 24..25: byte-address swizzle of the staged run (3, 2 or 0).  (24-bit products and
                                 // 16-bit compares take the width without a mask.)
  uint32_t byte_off;             // LDS byte address of the group's first packed word
};

template <int DT, int LPG_LOG2, int DIV = 1>
struct alignas(16) WaveLds {
  using S = TileShape<DT, LPG_LOG2, DIV>;
  // First the complemented random bytes of the tile (byte e serves tile element e); once every lane has
  // taken its bytes into registers the same memory stages the tile's packed words (at most
  // 8 bits per element, so the run always fits).
  // The staged run starts up to three words in, so that 16-byte pieces of it line up with
  // 16-byte pieces of the packed buffer.
  union {
    uint8_t rand_bytes[S::kElems];
    uint32_t stage[S::kElems / 4 + 4];
  };
  GroupInfo info[kWave];
  float2 stat[kWave];                   // (min, max) per group, written by the group's last lane;
                                        // later (metrics variant) the group's (error, magnitude) sums
  float gscale[kWave];                  // scale per group (metrics variant)
  float gvar[kWave];                    // sum of T*(256-T) per group (metrics variant)
};

// ---- the tile in which a tensor ends ---------------------------------------------------------
// A tensor rarely ends with a whole tile.  What is left, whole groups and at last a short one, is one more tile whose
// chunks past the end hold copies of the tensor's last element: they leave the short group's minimum and maximum as
// they are, and their codes are taken out of the last packed word again (end_run).  The groups
// used to go one by one through quantize_pack_group_body in a workgroup of their own, up to 63 chains of
// dependent loads of ~3 us each behind four waves: 6774528 bfloat16 elements, groups of 64, three widths, both directions
// 52.7 us, now 13.4.
// `len` elements, 1 <= len < LOADS * kWave * kEpl, from `chunks` on; chunk u * kWave + lane goes to raw[u].
template <int DT, int LOADS>
__device__ __forceinline__ void short_tile_load(const u32x4* chunks, int len, int lane, uint4 (&raw)[LOADS]) {
  constexpr int kEpl = ElemTraits<DT>::kPerLoad;
  const int whole = len / kEpl, last = len - 1;
  // every load is issued before any is used, that of the last elements behind the chunks
  u32x4 v[LOADS];
#pragma unroll
  for (int u = 0; u < LOADS; ++u) v[u] = u32x4{0u, 0u, 0u, 0u};
  if (whole > 0) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const int c = u * kWave + lane;
      v[u] = __builtin_nontemporal_load(&chunks[c < whole ? c : whole - 1]);
    }
  }
  // The chunk the tensor ends in, behind its end the last element: an element per lane, handed out as scalars (the same in all
  // lanes they took a register per element, which is what made whole tiles spill beside this).
  const int i = min(whole * kEpl + (lane & (kEpl - 1)), last);
  const uint32_t elem = DT == kF32 ? reinterpret_cast<const uint32_t*>(chunks)[i] : reinterpret_cast<const uint16_t*>(chunks)[i];
  auto of = [&](int e) { return (uint32_t)__builtin_amdgcn_readlane((int)elem, e); };
  uint32_t edge[4], end = of(kEpl - 1);              // fewer than kEpl are left: the last element
  if (DT != kF32) end |= end << 16;
#pragma unroll
  for (int e = 0; e < 4; ++e) edge[e] = DT == kF32 ? of(e) : of((2 * e) % kEpl) | (of((2 * e + 1) % kEpl) << 16);
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int c = u * kWave + lane;
    raw[u] = make_uint4(v[u].x, v[u].y, v[u].z, v[u].w);
    if ((u + 1) * kWave > whole) {                   // (the whole wave)
      if (c == whole) raw[u] = make_uint4(edge[0], edge[1], edge[2], edge[3]);
      if (c > whole) raw[u] = make_uint4(end, end, end, end);
    }
  }
}
// The first `len` elements of such a tile to `chunks`.
template <int DT, int LOADS>
__device__ __forceinline__ void short_tile_store(u32x4* chunks, int len, int lane, const uint4 (&raw)[LOADS]) {
  constexpr int kEpl = ElemTraits<DT>::kPerLoad;
  const int whole = len / kEpl, rest = len % kEpl;
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int c = u * kWave + lane;
    if (c < whole) {
      chunks[c] = u32x4{raw[u].x, raw[u].y, raw[u].z, raw[u].w};
    } else if (c == whole) {
      const uint32_t w[4] = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
#pragma unroll
      for (int e = 0; e < kEpl; ++e) {
        if (e >= rest) continue;
        if (DT == kF32) reinterpret_cast<uint32_t*>(chunks)[c * kEpl + e] = w[e % 4];
        else reinterpret_cast<uint16_t*>(chunks)[c * kEpl + e] = (uint16_t)(w[e / 2] >> (16 * (e & 1)));
      }
    }
  }
}

// Codes of one 16-byte chunk, one to a byte (code_bytes): q[0] elements 0..3, q[1] elements 4..7 (16-bit inputs).
// not_rnd: the complements of the chunk's random bytes, one dword per four elements.
//
// METRICS: also returns this lane's share of the group's importance sums (Sec. 3.2 names
// quantization error and tensor magnitude): err += (x - xhat)^2 with xhat = fma(code, scale, mn)
// as the dequantizer computes it, mag += x^2, both in binary32; var = sum of T*(256-T), the
// variance of the stochastic rounding in units of scale^2 / 65536 (exact integer).
//
// Elements from `valid` on (SHORT: the tensor ends in this chunk or before it) count for no sum.
//
// A chunk comes in its loaded form.  binary16 without metrics is never widened: min - x is
// one mixed-precision fma per element.  With metrics the values that the
// statistics widened would hold twice the registers until here, so they are made again (the empty statement keeps the
// compiler from keeping the first ones): 128 -> 96 registers, 4 -> 5 waves per SIMD, 361 M bfloat16 elements, groups of 64,
// call with selection and plan 285 -> 279 us.  AGAIN: the same without metrics.  Tiles of bfloat16 keep them (93 M elements,
// groups of 256, 2 bits, both directions, 4 waves with kept values 70.3 us, 5 waves with values made again 71.9; other
// widths 0.995 to 1.01 of each other), units make them again, at 5 waves: the same within 1 % (24 tensors of rows of 768 and 3072 in list
// calls, kept / made again {2,4,8} 76.3 / 75.8 us, 8 bits 78.9 / 78.5, 2 bits 65.8 / 66.3, 46 M elements in groups of 768, four
// widths, 49.7 / 49.0).
template <int DT, bool EXACT2, bool METRICS = false, bool SHORT = false, bool AGAIN = false>
__device__ __forceinline__ void quantize_raw_chunk(uint4& raw, float mn, float invs, const uint32_t* not_rnd,
                                                   uint32_t (&q)[ElemTraits<DT>::kPerLoad / 4], int valid = 8,
                                                   float scale = 0.0f, float* err = nullptr, float* mag = nullptr,
                                                   float* var = nullptr) {
  constexpr int kEpl = ElemTraits<DT>::kPerLoad;
  if ((METRICS || AGAIN) && DT != kF32) asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
  int t[kEpl];
#pragma unroll
  for (int e = 0; e < kEpl; ++e) {
    float d;
    if constexpr (DT == kF16 && !METRICS) d = (e & 1) ? min_minus_half<1>(w[e >> 1], mn) : min_minus_half<0>(w[e >> 1], mn);
    else d = mn - chunk_elem<DT>(raw, e);
    t[e] = neg_position<EXACT2>(d, invs);
  }
  if constexpr (kEpl == 4) q[0] = code_bytes(t, not_rnd[0]);
  else code_bytes(t, not_rnd[0], not_rnd[1], q[0], q[kEpl / 4 - 1]);
  if constexpr (METRICS) {
    float e2 = 0.0f, m2 = 0.0f;
    uint32_t t_sum = 0u, t_sq = 0u;
#pragma unroll
    for (int c = 0; c < kEpl / 4; ++c) {
      int rt[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = !SHORT || c * 4 + e < valid;
        rt[e] = in ? t[c * 4 + e] : 0;
        if (in) {
          const float xv = chunk_elem<DT>(raw, c * 4 + e);
          const float d = xv - __builtin_fmaf((float)((q[c] >> (24 - 8 * e)) & 0xFFu), scale, mn);
          e2 = __builtin_fmaf(d, d, e2);
          m2 = __builtin_fmaf(xv, xv, m2);
        }
      }
      sr_variance_sums(rt, t_sum, t_sq);
    }
    *err = e2;
    *mag = m2;
    *var = (float)(256u * t_sum - t_sq);
  }
}
// The last word of a run that ends with a short group, of `bits` bits: what the codes of the copies behind the tensor's last
// element (short_tile_load) left in it becomes 0.
__device__ __forceinline__ void end_run(uint32_t* last_word, uint32_t bits, int lane) {
  if ((bits & 31u) != 0u && lane == 0) *last_word &= ~0u << (32u - (bits & 31u));
  wave_lds_sync();
}

// binary16 tiles: one [-max : min] dword (two binary16 halves, daf_device.h) per (load, lane run)
// segment in stat[segment].x; nothing is widened.
template <int LPG_LOG2, int DIV>
__device__ __forceinline__ void tile_minmax_f16(const uint4 (&raw)[TileShape<kF16, LPG_LOG2, DIV>::kLoads], float2* stat,
                                                int lane) {
  using S = TileShape<kF16, LPG_LOG2, DIV>;
  static_assert(S::kLoads % 4 == 0, "loads are reduced four at a time");
#pragma unroll
  for (int u = 0; u < S::kLoads; u += 4) {
    uint32_t p[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) p[h] = chunk_stat_f16(raw[u + h]);
    seg_pk_min_x4<S::kLaneLog2>(p[0], p[1], p[2], p[3]);
    if ((lane & (S::kLpg - 1)) == S::kLpg - 1) {
#pragma unroll
      for (int h = 0; h < 4; ++h) stat[(u + h) * S::kGpl + (lane >> S::kLaneLog2)].x = u2f(p[h]);
    }
  }
}

// Leaves one (min, max) pair per (load, lane run) segment in stat[load * runs_per_load + run]; a group's
// segments are consecutive entries.
template <int DT, int LPG_LOG2, int DIV = 1>
__device__ __forceinline__ void tile_minmax(const uint4 (&raw)[TileShape<DT, LPG_LOG2, DIV>::kLoads], float2* stat, int lane) {
  using S = TileShape<DT, LPG_LOG2, DIV>;
  constexpr int kEpl = S::kEpl;
  float xf[S::kLoads][kEpl];
  static_assert(S::kLoads % 2 == 0, "loads are reduced in pairs");
  if constexpr (DT == kF32 && LPG_LOG2 >= 5 && S::kLoads == 16) {
    // groups of 32 or 64 lanes: all 16 loads are reduced together (transposed reduction)
    float lmn[16], lmx[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
#pragma unroll
      for (int e = 0; e < kEpl; ++e) xf[u][e] = chunk_elem<DT>(raw[u], e);
      lmn[u] = vmin(vmin3(xf[u][0], xf[u][1], xf[u][2]), xf[u][3]);
      lmx[u] = vmax(vmax3(xf[u][0], xf[u][1], xf[u][2]), xf[u][3]);
    }
    float mn[2], mx[2];
    transposed_minmax16<S::kLaneLog2>(lmn, lmx, mn, mx);
    if ((lane & 3) == 0) {
      if (LPG_LOG2 >= 6) {
        stat[(lane >> 2) & 15] = make_float2(mn[0], mx[0]);
      } else {
        const int u = (lane >> 2) & 7, seg = lane >> 5;
        stat[u * 2 + seg] = make_float2(mn[0], mx[0]);
        stat[(u + 8) * 2 + seg] = make_float2(mn[1], mx[1]);
      }
    }
  } else {
    // two loads at a time so that four independent DPP chains interleave
#pragma unroll
    for (int u = 0; u < S::kLoads; u += 2) {
      float mn[2], mx[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int e = 0; e < kEpl; ++e) xf[u + h][e] = chunk_elem<DT>(raw[u + h], e);
        const float(&v)[kEpl] = xf[u + h];
        if (kEpl == 4) {
          mn[h] = vmin(vmin3(v[0], v[1], v[2]), v[3]);
          mx[h] = vmax(vmax3(v[0], v[1], v[2]), v[3]);
        } else {
          mn[h] = vmin(vmin3(vmin3(vmin3(v[0], v[1], v[2]), v[3], v[4 % kEpl]), v[5 % kEpl], v[6 % kEpl]), v[7 % kEpl]);
          mx[h] = vmax(vmax3(vmax3(vmax3(v[0], v[1], v[2]), v[3], v[4 % kEpl]), v[5 % kEpl], v[6 % kEpl]), v[7 % kEpl]);
        }
      }
      seg_minmax_x2<S::kLaneLog2>(mn[0], mx[0], mn[1], mx[1]);
      if ((lane & (S::kLpg - 1)) == S::kLpg - 1) {
        stat[u * S::kGpl + (lane >> S::kLaneLog2)] = make_float2(mn[0], mx[0]);
        stat[(u + 1) * S::kGpl + (lane >> S::kLaneLog2)] = make_float2(mn[1], mx[1]);
      }
    }
  }
}

// The stores of one chunk where the width differs from lane to lane: all four follow each other, each under its lanes' mask.
// (From conditions the compiler makes a tree of branches, 20 scalar instructions and up to six jumps a chunk: 25 M binary16 elements,
// four widths, both directions 26.7 us with it, 26.0 so; 361 M bfloat16 elements 316 / 314, with metrics and selection 260 / 258.)  `width`: its lower
// 16 bits.  EPL 4: of 1-bit codes only the even lanes store.
// (The wait states at the end: a DPP instruction may follow a vector write of EXEC after five.)
template <int EPL>
__device__ __forceinline__ void store_by_width(uint32_t addr, uint32_t width, uint32_t q0, uint32_t q1, uint32_t w4, uint32_t w2,
                                               uint32_t w1) {
  uint64_t all;
  if constexpr (EPL == 4) {
    asm volatile("s_mov_b64 %0, exec\n"
                 "v_cmpx_eq_u16 vcc, 8, %2\n ds_write_b32 %1, %3\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 4, %2\n ds_write_b16 %1, %4\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 2, %2\n ds_write_b8 %1, %5\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 1, %2\n s_and_b64 exec, exec, %7\n ds_write_b8 %1, %6\n s_mov_b64 exec, %0\n s_nop 2"
                 : "=&s"(all)
                 : "v"(addr), "v"(width), "v"(q0), "v"(w4), "v"(w2), "v"(w1), "s"(0x5555555555555555ull)
                 : "memory", "vcc", "scc");
  } else {
    const uint64_t q = ((uint64_t)q1 << 32) | q0;
    asm volatile("s_mov_b64 %0, exec\n"
                 "v_cmpx_eq_u16 vcc, 8, %2\n ds_write_b64 %1, %3\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 4, %2\n ds_write_b32 %1, %4\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 2, %2\n ds_write_b16 %1, %5\n s_mov_b64 exec, %0\n"
                 "v_cmpx_eq_u16 vcc, 1, %2\n ds_write_b8 %1, %6\n s_mov_b64 exec, %0\n s_nop 2"
                 : "=&s"(all)
                 : "v"(addr), "v"(width), "v"(q), "v"(w4), "v"(w2), "v"(w1)
                 : "memory", "vcc", "scc");
  }
}

// Drops the codes of one chunk (bytes, as quantize_raw_chunk returns them) at LDS byte address `addr` of the staged word run: a
// nibble pair, a byte, a halfword or whole words.  PER_LANE: `b` differs from lane to lane, and only its lower 16 bits count.
template <int EPL, bool PER_LANE>
__device__ __forceinline__ void stage_chunk(uint32_t addr, uint32_t b, const uint32_t (&q)[EPL / 4], int lane) {
  typedef __attribute__((address_space(3))) uint8_t lds_u8;
  uint8_t* at = (uint8_t*)(lds_u8*)(uintptr_t)addr;
  if constexpr (EPL == 4) {
    // 1 bit: the even lane takes its odd neighbour's nibble
    auto nibbles = [&] {
      const uint32_t bits = pack_codes<1>(q[0]), nb = dpp<kDppXor1>(bits, bits);
      return (bits << 4) | nb;
    };
    if constexpr (PER_LANE) {
      store_by_width<EPL>(addr, b, q[0], 0u, pack_codes<4>(q[0]), pack_codes<2>(q[0]), nibbles());
    } else if (b == 1u) {
      const uint32_t both = nibbles();
      if ((lane & 1) == 0) *at = (uint8_t)both;
    } else if (b == 2u) {
      *at = (uint8_t)pack_codes<2>(q[0]);
    } else if (b == 4u) {
      *reinterpret_cast<uint16_t*>(at) = (uint16_t)pack_codes<4>(q[0]);
    } else {
      *reinterpret_cast<uint32_t*>(at) = q[0];
    }
  } else {
    const uint32_t q0 = q[0], q1 = q[EPL / 4 - 1];
    if constexpr (PER_LANE) {
      store_by_width<EPL>(addr, b, q0, q1, pack_codes<4>(q0, q1), pack_codes<2>(q0, q1), pack_codes<1>(q0, q1));
    } else if (b == 8u) {
      *reinterpret_cast<uint2*>(at) = make_uint2(q0, q1);
    } else if (b == 4u) {
      *reinterpret_cast<uint32_t*>(at) = pack_codes<4>(q0, q1);
    } else if (b == 2u) {
      *reinterpret_cast<uint16_t*>(at) = (uint16_t)pack_codes<2>(q0, q1);
    } else {
      *at = (uint8_t)pack_codes<1>(q0, q1);
    }
  }
}

// The (min, max) of n <= kMaxFold pairs, by all kThreads threads of a workgroup; every thread has the result.
constexpr int kFoldPerThread = 8, kMaxFold = kFoldPerThread * kThreads;
__device__ __forceinline__ float2 fold_pairs(const float2* __restrict__ pairs, int n) {
  __shared__ float2 wave_pair[kWavesPerBlock];
  float2 p[kFoldPerThread];
#pragma unroll
  for (int j = 0; j < kFoldPerThread; ++j) {
    const int i = j * kThreads + (int)threadIdx.x;
    p[j] = pairs[i < n ? i : n - 1];
  }
  float mn = vmin3(p[0].x, p[1].x, p[2].x), mn2 = p[3].x, mx = vmax3(p[0].y, p[1].y, p[2].y), mx2 = p[3].y;
#pragma unroll
  for (int j = 4; j < kFoldPerThread; j += 2) {
    mn = vmin(mn, p[j].x); mx = vmax(mx, p[j].y);
    mn2 = vmin(mn2, p[j + 1].x); mx2 = vmax(mx2, p[j + 1].y);
  }
  seg_minmax_x2<6>(mn, mx, mn2, mx2);
  if ((threadIdx.x & (kWave - 1)) == kWave - 1) wave_pair[threadIdx.x >> 6] = make_float2(vmin(mn, mn2), vmax(mx, mx2));
  __syncthreads();
  float2 r = wave_pair[0];
#pragma unroll
  for (int w = 1; w < kWavesPerBlock; ++w) {
    r.x = vmin(r.x, wave_pair[w].x);
    r.y = vmax(r.y, wave_pair[w].y);
  }
  return r;
}

// B = 1, 2, 4, 8: every group has that width (offsets are computed).  B = 0: per-group widths
// from `bits`, offsets from `off`.
// One tile per wave; the hardware schedules the waves.  (A looping variant in which a wave
// prefetched its next tile while quantizing the current one was slower: it needs more
// registers, and on this architecture loads and stores share one in-order counter, so waiting
// for a prefetched load also waits for the stores issued after it.)
//
// EXT = true (only with the one-group-per-tile shape): the group is `tiles_per_group` tiles
// long and its (min, max) comes from `ext_stat`, computed by an earlier pass; the tile skips
// the reduction, and the group's first tile stores min and scale.
//
// METRICS = true: additionally writes, per group, the sums (x - xhat)^2 and x^2 over the group
// (binary32, accumulated per lane, then across the group's lanes, then across its loads) and the
// variance of the stochastic rounding, scale^2 * sum p (1 - p).
//
// RELU = true: x holds z; every element becomes max(z, +0) right after the load, the result is
// written to out_y in the same layout (out_y may be x itself: a lane only overwrites chunks it
// has already loaded), and everything else sees y.
//
// SHORT: the tile in which the tensor ends; it holds `len` elements (short_tile_load).
//
// FOLD (with EXT, one group for the tensor): ext_stat holds n_ext (min, max) pairs that every workgroup reduces for
// itself, behind the tile's loads; all its waves take part (fold_pairs has a barrier).
// (The LDS of a workgroup: one place for a kernel's whole and short tiles.)
template <int DT, int LPG_LOG2, int DIV>
__device__ __forceinline__ WaveLds<DT, LPG_LOG2, DIV>* tile_lds() {
  __shared__ WaveLds<DT, LPG_LOG2, DIV> all[kWavesPerBlock];
  return all;
}

template <int DT, int LPG_LOG2, int B, bool EXT = false, bool METRICS = false, bool RELU = false, int DIV = 1,
          bool FOLD = false, bool SHORT = false>
__device__ __forceinline__ void quantize_pack_tile_body(
    typename std::conditional<RELU, const u32x4*, const u32x4* __restrict__>::type x, int64_t tile, int wave_in_block,
    const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t* __restrict__ words, float* __restrict__ out_min, float* __restrict__ out_scale,
    const float2* __restrict__ ext_stat, int64_t tiles_per_group, float* __restrict__ out_metrics,
    u32x4* out_y, int n_ext = 0, int len = 0) {
  using S = TileShape<DT, LPG_LOG2, DIV>;
  static_assert(!FOLD || EXT, "pairs are folded for external statistics");
  static_assert(!EXT || S::kGroups == 1, "external statistics: the tile is part of one group");
  static_assert(!(EXT && METRICS), "metrics are not computed for groups longer than a tile");
  static_assert(!METRICS || S::kLoads % 2 == 0, "the metrics' sums over the lanes are taken two loads at a time");
  static_assert(!(RELU && (EXT || METRICS)), "the fused max(z, 0) exists for the plain tile kernel only");
  static_assert(!(SHORT && EXT), "a short tile holds whole groups and the tensor's last");
  constexpr int kEpl = S::kEpl;
  constexpr bool kMixed = (B == 0);
  constexpr uint32_t kGroupWords32 = S::kGroupSize / 32;      // words per group and bit of width

  const int lane = threadIdx.x & (kWave - 1);
  WaveLds<DT, LPG_LOG2, DIV>& lds = tile_lds<DT, LPG_LOG2, DIV>()[wave_in_block];
  const uint32_t lane_in_run = (uint32_t)(lane & (S::kLpg - 1));
  // LDS byte address of the staging area (16-byte aligned, so the byte swizzles commute with it)
  const uint32_t stage_base = (uint32_t)reinterpret_cast<uintptr_t>(lds.stage);
  // groups of the tile, and the length of the last one
  const int n_groups = SHORT ? (len + S::kGroupSize - 1) / S::kGroupSize : S::kGroups;
  const uint32_t last_len = SHORT ? (uint32_t)(len - (n_groups - 1) * S::kGroupSize) : (uint32_t)S::kGroupSize;

  // 1. all global loads of the tile, issued up front
  uint4 raw[S::kLoads];
  if constexpr (SHORT) {
    short_tile_load<DT>(&x[tile * (S::kLoads * kWave)], len, lane, raw);
  } else {
#pragma unroll
    for (int u = 0; u < S::kLoads; ++u) {
      const u32x4 v = __builtin_nontemporal_load(&x[tile * (S::kLoads * kWave) + u * kWave + lane]);
      raw[u] = make_uint4(v.x, v.y, v.z, v.w);
    }
  }
  if constexpr (RELU) {
#pragma unroll
    for (int u = 0; u < S::kLoads; ++u) {
      raw[u] = make_uint4(relu_bits<DT>(raw[u].x), relu_bits<DT>(raw[u].y), relu_bits<DT>(raw[u].z),
                          relu_bits<DT>(raw[u].w));
      const u32x4 y = {raw[u].x, raw[u].y, raw[u].z, raw[u].w};
      if (!SHORT) out_y[tile * (S::kLoads * kWave) + u * kWave + lane] = y;    // the next layer reads it soon: cached store
    }
    if constexpr (SHORT) short_tile_store<DT>(&out_y[tile * (S::kLoads * kWave)], len, lane, raw);
  }

  {
    // first group of the tile, and the tile's position inside it (EXT only)
    const int64_t g0 = EXT ? tile / tiles_per_group : tile * S::kGroups;
    const uint32_t tile_in_group = EXT ? (uint32_t)(tile - g0 * tiles_per_group) : 0u;

    uint32_t my_b = (uint32_t)B;
    uint32_t tile_base;
    if (kMixed) {
      my_b = (lane < n_groups) ? (uint32_t)bits[g0 + lane] : 1u;
      tile_base = off[g0];
      if (EXT) tile_base += tile_in_group * (kGroupWords32 * (uint32_t)__builtin_amdgcn_readfirstlane((int)my_b));
    } else {
      tile_base = (uint32_t)tile * (uint32_t)(S::kGroups * kGroupWords32 * B);
    }

    // The run is staged `head` words into the staging area, head = the word index of its first
    // word in the packed buffer modulo 4: 16-byte pieces of the two then coincide.
    const uint32_t head = ((uint32_t)(reinterpret_cast<uintptr_t>(words) >> 2) + tile_base) & 3u;

    // 2. random bytes of the tile, complemented (independent of the data; overlaps the loads' latency)
    {
      constexpr int kBlocks = S::kElems / kElemsPerPhilox;
      static_assert((kBlocks & (kBlocks - 1)) == 0, "a tile's block numbers agree in their upper halves");
      const uint64_t blk0 = (uint64_t)tile * kBlocks;
      uint4* dst = reinterpret_cast<uint4*>(lds.rand_bytes);
#pragma unroll
      for (int m = 0; m < S::kPhilox; ++m)
        dst[m * kWave + lane] = philox_block<true>((uint32_t)blk0 + (uint32_t)(m * kWave + lane), (uint32_t)(blk0 >> 32), seed_lo, seed_hi);
    }

    // 3. per-group min/max: in-lane over the chunk, then across the group's lanes.
    //    binary16 tiles: packed minimum / maximum on the loaded pairs, and
    //    the subtraction of step 5 widens on the fly.
    constexpr bool kPairs16 = DT == kF16;
    if constexpr (!EXT) {
      if constexpr (kPairs16) tile_minmax_f16<LPG_LOG2, DIV>(raw, lds.stat, lane);
      else tile_minmax<DT, LPG_LOG2, DIV>(raw, lds.stat, lane);
    }
    wave_lds_sync();

    // 4. lane g of the wave finishes group g of the tile: scale, reciprocal, place in the run
    bool need_exact2;
    uint32_t tile_words;
    [[maybe_unused]] uint32_t last_bits;        // of the short group
    {
      float2 st;
      if constexpr (FOLD) {
        st = fold_pairs(ext_stat, n_ext);
      } else if constexpr (EXT) {
        st = ext_stat[g0];
      } else if constexpr (kPairs16) {
        uint32_t pk = f2u(lds.stat[(lane & (S::kGroups - 1)) * S::kLoadsPerGroup].x);
#pragma unroll
        for (int j = 1; j < S::kLoadsPerGroup; ++j)
          pk = pk_min_f16(pk, f2u(lds.stat[(lane & (S::kGroups - 1)) * S::kLoadsPerGroup + j].x));
        st = make_float2(stat_f16_min(pk), stat_f16_max(pk));
      } else {
        // the group's (load, lane run) segments are consecutive entries of stat
        st = lds.stat[(lane & (S::kGroups - 1)) * S::kLoadsPerGroup];
#pragma unroll
        for (int j = 1; j < S::kLoadsPerGroup; ++j) {
          const float2 t = lds.stat[(lane & (S::kGroups - 1)) * S::kLoadsPerGroup + j];
          st.x = vmin(st.x, t.x);
          st.y = vmax(st.y, t.y);
        }
      }
      const GroupScale s = group_scale(st.x, st.y, my_b);
      const float invs = s.inv * kScale;
      // (the variant with two multiplications is right for every group: short tiles have it alone)
      need_exact2 = SHORT || __builtin_amdgcn_ballot_w64(!(invs <= 3.402823466e+38f) && lane < S::kGroups) != 0ull;
      uint32_t woff;
      if (kMixed) {
        const uint32_t w = (lane < S::kGroups) ? kGroupWords32 * my_b : 0u;
        const uint32_t incl = wave_inclusive_sum(w);
        tile_words = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        woff = incl - w;
      } else {
        tile_words = S::kGroups * kGroupWords32 * B;
        woff = (uint32_t)lane * (kGroupWords32 * B);
      }
      // (a short tile's run is laid out in LDS as if all its groups were there and whole; what leaves ends early)
      if constexpr (SHORT) {
        last_bits = last_len * (uint32_t)__builtin_amdgcn_readlane((int)my_b, n_groups - 1);
        tile_words = (uint32_t)__builtin_amdgcn_readlane((int)woff, n_groups - 1) + ((last_bits + 31u) >> 5);
      }
      if (lane < S::kGroups) {
        if ((!EXT || tile_in_group == 0u) && (!SHORT || lane < n_groups)) {
          if (kMixed) {
            // Streaming stores: with many packed words per tile (wide codes) plain stores
            // of these two small runs slowed the whole kernel down measurably; with the
            // few words of uniform narrow codes they made no difference.
            __builtin_nontemporal_store(s.mn, &out_min[g0 + lane]);
            __builtin_nontemporal_store(s.scale, &out_scale[g0 + lane]);
          } else {
            out_min[g0 + lane] = s.mn;
            out_scale[g0 + lane] = s.scale;
          }
        }
        GroupInfo gi;
        gi.mn = s.mn;
        gi.invs = need_exact2 ? s.inv : invs;
        // A lane's bits are written as a byte (swizzle 3), a halfword (2) or whole words (0).
        const uint32_t lane_bits = (uint32_t)kEpl * my_b;
        const uint32_t swz = (lane_bits <= 8u) ? 3u : (lane_bits == 16u) ? 2u : 0u;
        gi.b = my_b | (swz << 24);
        gi.byte_off = stage_base + (woff + head) * 4u;
        lds.info[lane] = gi;
        if (METRICS) lds.gscale[lane] = s.scale;
      }
      if (METRICS && S::kLoadsPerGroup > 1) {
        wave_lds_sync();                       // every lane has read its (min, max) pairs
        lds.stat[lane] = make_float2(0.0f, 0.0f);
        lds.gvar[lane] = 0.0f;
      }
    }

    // the lane's random bytes, one dword per four elements, out of LDS before it is reused
    uint32_t rnd[S::kLoads][kEpl / 4];
#pragma unroll
    for (int u = 0; u < S::kLoads; ++u) {
      if (kEpl == 4) {
        rnd[u][0] = reinterpret_cast<const uint32_t*>(lds.rand_bytes)[u * kWave + lane];
      } else {
        const uint2 r2 = reinterpret_cast<const uint2*>(lds.rand_bytes)[u * kWave + lane];
        rnd[u][0] = r2.x;
        rnd[u][kEpl / 4 - 1] = r2.y;
      }
    }
    wave_lds_sync();

    // 5. quantize every chunk and drop its bits at their place in the staged word run.
    //    The staged run is a big-endian bit string per word: byte k of the string lives at
    //    byte address k^3, halfword k at byte address 2k^2.
    //    (One copy of the loop per multiplication variant, chosen once per tile: the variant for
    //    groups whose reciprocal times 256 overflows is rare.)
    auto quantize_tile = [&](auto exact2) {
      constexpr bool kExact2 = decltype(exact2)::value;
      // (what the two copies have in common would be computed before the branch, a register more than there are)
      if (METRICS && DT == kF16 && kExact2) asm volatile("" ::: "memory");
      [[maybe_unused]] float metric_sums[2][3];  // error, magnitude, variance of the last two loads
#pragma unroll
      for (int u = 0; u < S::kLoads; ++u) {
        const int grp = (u * S::kGpl + (lane >> S::kLaneLog2)) / S::kLoadsPerGroup;
        // position of this lane's chunk among the chunks of its group
        const uint32_t lig = lane_in_run + (uint32_t)(u % S::kLoadsPerGroup) * kWave;
        float g_mn, g_invs;
        uint32_t b, addr;
        if (kMixed) {
          const GroupInfo gi = lds.info[grp];
          g_mn = gi.mn; g_invs = gi.invs; b = gi.b;
          // byte address of this lane's bits: lig * (kEpl*b) bits = lig*b*kEpl/8 bytes
          addr = (gi.byte_off + (kEpl == 8 ? __umul24(lig, gi.b) : __umul24(lig, gi.b) >> 1)) ^ (gi.b >> 24);
        } else {
          const float2 mi = *reinterpret_cast<const float2*>(&lds.info[grp]);
          g_mn = mi.x; g_invs = mi.y; b = B;
          constexpr uint32_t kLaneBits = (uint32_t)kEpl * B;
          constexpr uint32_t kSwz = (kLaneBits <= 8u) ? 3u : (kLaneBits == 16u) ? 2u : 0u;
          addr = (stage_base + head * 4u + (uint32_t)grp * (kGroupWords32 * B * 4u) + ((lig * kLaneBits) >> 3)) ^ kSwz;
        }
        uint32_t q[kEpl / 4];
        [[maybe_unused]] const int valid = SHORT ? len - (u * kWave + lane) * kEpl : 8;         // elements from here to the end
        if constexpr (METRICS) {
          const float g_scale = lds.gscale[grp];
          float* sums = metric_sums[u & 1];
          quantize_raw_chunk<DT, kExact2, true, SHORT>(raw[u], g_mn, g_invs, rnd[u], q, valid, g_scale, &sums[0],
                                                       &sums[1], &sums[2]);
          if (u & 1) {                           // over the group's lanes, two loads at a time
            seg_sum6<S::kLaneLog2>(metric_sums[0], metric_sums[1]);
            if (lane_in_run == (uint32_t)S::kLpg - 1u) {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                const int gh = ((u - 1 + h) * S::kGpl + (lane >> S::kLaneLog2)) / S::kLoadsPerGroup;
                const float* r = metric_sums[h];
                if (S::kLoadsPerGroup == 1) {
                  lds.stat[gh] = make_float2(r[0], r[1]);
                  lds.gvar[gh] = r[2];
                } else {
                  const float2 acc = lds.stat[gh];    // the group's earlier loads (same lane, in order)
                  lds.stat[gh] = make_float2(acc.x + r[0], acc.y + r[1]);
                  lds.gvar[gh] += r[2];
                }
              }
            }
          }
        } else {
          quantize_raw_chunk<DT, kExact2, false, SHORT>(raw[u], g_mn, g_invs, rnd[u], q);
        }
        // (a load's 64 lanes are of one group: its width is a scalar)
        constexpr bool kPerLane = kMixed && S::kLaneLog2 < 6;
        stage_chunk<kEpl, kPerLane>(addr, kMixed && !kPerLane ? (uint32_t)__builtin_amdgcn_readfirstlane((int)b) & 0xFFu : b, q, lane);
      }
    };
    if (need_exact2) quantize_tile(std::true_type{});
    else             quantize_tile(std::false_type{});
    wave_lds_sync();
    if constexpr (SHORT) end_run(&lds.stage[head + tile_words - 1u], last_bits, lane);

    // 6. the tile's words are one contiguous run of the packed buffer; they leave in 16-byte
    //    pieces (single words at a ragged start or end) with streaming stores: the words are read
    //    back by the backward pass, long after they have left the caches (with ordinary stores
    //    the mixed-width kernels ran a tenth slower).
    {
      const uint32_t span = head + tile_words;
      uint32_t* dst = words + tile_base - head;                 // 16-byte aligned
      const uint32_t full_begin = (head + 3u) & ~3u, full_end = span & ~3u;
      for (uint32_t w0 = full_begin + (uint32_t)lane * 4u; w0 < full_end; w0 += kWave * 4u)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(&lds.stage[w0]), reinterpret_cast<u32x4*>(dst + w0));
      // the up to three words before the first and after the last whole piece: lanes 0..3 and 4..7
      const uint32_t w = (lane < 4) ? (uint32_t)lane : full_end + (uint32_t)lane - 4u;
      // (the run of a short tile may end before its first whole piece begins)
      if (lane < 8 && ((lane < 4) ? (w >= head && w < full_begin && (!SHORT || w < span))
                                  : (w < span && (!SHORT || w >= full_begin))))
        __builtin_nontemporal_store(lds.stage[w], dst + w);
    }
    if constexpr (METRICS) {
      // (the lane counted anew: its addresses from step 4 would hold registers until here)
      const int g = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
      if (g < n_groups) {
        const float sc = lds.gscale[g];
        float* m = out_metrics + 3 * (g0 + g);
        m[0] = lds.stat[g].x;
        m[1] = lds.stat[g].y;
        m[2] = (lds.gvar[g] * 1.52587890625e-05f) * (sc * sc);
      }
    }
  }
}

// Waves per SIMD of the tile kernel.  At least: as many as the whole tiles' registers allow without spilling; the short tile's
// code shall not cost a wave (metrics, 361 M bfloat16 elements, groups of 64: 4 waves instead of 3, 311 -> 285 us, whole call).
// Metrics in 16-bit formats: 5, without a spill (binary16, 361 M elements, groups of 64, 5 waves with spills / without / 4 waves:
// 294 / 288 / 294 us; 180 M, groups of 128 151.2 / 149.9 / 151.3, of 256 149.3 / 148.2 / 148.9; the middle
// one moves by card, in groups of 128 and 256 from 2 % ahead of the first to 4 % behind it).
// At most: more waves than these scatter the streams of a binary32 tensor (both directions, 47 M elements, 2 bits, 4 / 5 / 6 / 8
// waves: 70.3 / 69.1 / 67.1 / 68.0 us; 92 M, 8 bits: 158.5 / 157.0 / 159.7 / 160.9; as many as fit / at most these: relu 2 bits
// 147.4 / 145.5, relu four widths 152.8 / 150.9, 51 M elements, four widths 81.7 / 81.7, 94 M, {2,4,8} 151.5 / 149.7).
template <int DT, int LPG_LOG2, bool METRICS>
constexpr int tile_min_waves() {
  if (DT == kF32) return LPG_LOG2 == 10 ? 4 : 1;
  if (METRICS) return 5;
  return DT == kF16 ? (LPG_LOG2 == 2 ? 8 : 6) : (LPG_LOG2 == 2 ? 7 : 4);
}
template <int DT, int B, bool METRICS>
constexpr int tile_max_waves() {
  return DT != kF32 || METRICS ? 8 : B == 8 ? 5 : 6;
}

// LDS that a launch of `tiles` tiles asks for on top of the kernel's: as much as leaves four waves per SIMD where six fit.  Long runs of
// binary16 tiles are bound by HBM, and more waves than four scatter their streams, the more so the fewer instructions a wave has (2 bits
// took 2 to 6 % longer than before the codes became bytes).  Shorter ones want the waves.  Six / four, quantize alone: 25 M elements, groups of
// 128, four widths 14.0 / 15.1 us, 50 M 23.9 / 24.5, 72 M 32.2 / 32.6, 100 M 44.0 / 43.7, 2 bits 40.9 / 39.6; 200 M, groups of 1024, 2 bits 77.8 /
// 71.8, four widths 84.4 / 79.9; lists of 400 M elements, 2 bits, groups of 64 to 4096 2 to 8 % faster, 4 and 8
// bits the same; not those of 1 bit or several widths, from 5 % faster to 4 % slower by group size.  (Groups of 32 and the sums of
// metrics are bound by their instructions; with relu's output stored as well the same within 1 %, four widths in groups of 64 2 % slower: 119 M 103.1 /
// 105.7; the other formats' registers leave no more than six and four waves.)
constexpr int64_t kManyTiles = 6 << 12;                    // 101 M elements
template <int DT, int LPG_LOG2, bool METRICS = false, bool RELU = false>
unsigned tile_extra_lds(int64_t tiles) {
  if constexpr (DT == kF16 && LPG_LOG2 > 2 && !METRICS && !RELU) {
    constexpr unsigned kExtra = 12u << 10, kAll = kWavesPerBlock * sizeof(WaveLds<DT, LPG_LOG2, tile_div<DT, LPG_LOG2>()>) + kExtra;
    static_assert(4u * kAll <= (160u << 10) && 5u * kAll > (160u << 10), "four workgroups on a compute unit");
    return tiles > kManyTiles ? kExtra : 0u;
  }
  return 0u;
}

template <int DT, int LPG_LOG2, int B, bool EXT = false, bool METRICS = false, bool RELU = false, int DIV = 1>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(EXT ? 1 : tile_min_waves<DT, LPG_LOG2, METRICS>(), EXT ? 8 : tile_max_waves<DT, B, METRICS>())))
void k_quantize_pack_tile(
    typename std::conditional<RELU, const u32x4*, const u32x4* __restrict__>::type x, int64_t n_tiles,
    const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t* __restrict__ words, float* __restrict__ out_min, float* __restrict__ out_scale,
    const float2* __restrict__ ext_stat, int64_t tiles_per_group, float* __restrict__ out_metrics,
    u32x4* out_y, int short_len) {
  const int wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // The tile in which the tensor ends takes longer than a whole one and goes first, in a workgroup of its own: as the
  // grid's last wave it was the launch's end, and as the first of all it moved the others' tiles by one.
  const unsigned first_block = short_len > 0 ? 1u : 0u;
  if constexpr (!EXT) {
    if (blockIdx.x < first_block) {
      if (wave_in_block > 0) return;
      quantize_pack_tile_body<DT, LPG_LOG2, B, false, METRICS, RELU, DIV, false, true>(
          x, n_tiles, wave_in_block, bits, off, seed_lo, seed_hi, words, out_min, out_scale, nullptr, (int64_t)1, out_metrics,
          out_y, 0, short_len);
      return;
    }
  }
  const int64_t tile = (int64_t)(blockIdx.x - first_block) * kWavesPerBlock + wave_in_block;
  if (tile >= n_tiles) return;
  quantize_pack_tile_body<DT, LPG_LOG2, B, EXT, METRICS, RELU, DIV>(x, tile, wave_in_block, bits, off, seed_lo, seed_hi,
                                                                    words, out_min, out_scale, ext_stat,
                                                                    tiles_per_group, out_metrics, out_y);
}

// Several tensors in one launch (the activations a training step saves, Sec. 3.1): the tiles
// of all of them form one sequence, and a wave finds its tensor by walking the cumulative tile
// counts.  One launch has one ramp at its start and one tail at its end instead of one per
// tensor.  The descriptors travel as kernel arguments.
constexpr int kMaxBatch = 32;
struct BatchEntry {
  const void* x;
  const uint8_t* bits;
  const uint32_t* off;
  uint32_t* words;
  float* mn;
  float* sc;
  int32_t tile_end;                                 // tiles of this and all earlier entries
  int32_t short_len;                                // elements of the last of them where it is a short one, else 0
  uint32_t seed_lo, seed_hi;
};
static_assert(sizeof(BatchEntry) == 64, "a descriptor is one cache line");
struct Batch {
  uint32_t ends[kBatchSlots];                       // e[t].tile_end, 0xFFFFFFFF beyond n
  BatchEntry e[kMaxBatch];
  int32_t n;
  void clear() {
    n = 0;
    for (int i = 0; i < kBatchSlots; ++i) ends[i] = 0xFFFFFFFFu;
  }
};
static_assert(kMaxBatch <= kBatchSlots, "one cumulative count per entry");

// At most as many waves per SIMD as a single tensor's kernel has, in groups of 4096 three (17 tensors of 206 M elements, both
// directions, as many as fit / at most these: groups of 256, 2 bits 829.6 / 823.0 us, 8 bits 1021.9 / 1010.6, four widths
// 941.8 / 920.5; of 2048, 2 bits 841.9 / 843.2; of 4096, 1 bit 856.6 / 847.4, 2 bits 844.2 / 837.7, 4 bits 935.4 / 934.2, 8 bits
// 1011.6 / 1007.9, four widths 922.6 / 905.4).
template <int DT, int LPG_LOG2, int B>
constexpr int list_max_waves() {
  if (DT == kBF16 && LPG_LOG2 >= 5) return 4;                       // what all widths' registers allow, with short tiles and without
  return DT == kF32 && LPG_LOG2 == 10 ? 3 : tile_max_waves<DT, B, false>();
}
// SHORT: some tensors of the list end inside a tile.  Lists of whole tiles have the kernel without that code, and with it there
// shall be as many waves per SIMD as without.
template <int DT, int LPG_LOG2, int B, bool SHORT>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(SHORT && DT == kF16 ? 6 : 1, list_max_waves<DT, LPG_LOG2, B>())))
void k_quantize_pack_tile_batch(const Batch batch) {
  const int wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t gtile = (int64_t)blockIdx.x * kWavesPerBlock + wave_in_block;
  const int t = batch_entry_of(batch.ends, (uint32_t)gtile);
  if (t >= batch.n) return;                          // past the last tile (the grid is whole workgroups)
  const BatchEntry& e = batch.e[t];
  int64_t tile = gtile - (t ? batch.e[t - 1].tile_end : 0);
  if constexpr (SHORT) {
    if (e.short_len > 0 && --tile < 0) {             // a tensor's short tile goes first, as in k_quantize_pack_tile
      const int64_t last = e.tile_end - 1 - (t ? batch.e[t - 1].tile_end : 0);
      quantize_pack_tile_body<DT, LPG_LOG2, B, false, false, false, tile_div<DT, LPG_LOG2>(), false, true>(
          static_cast<const u32x4*>(e.x), last, wave_in_block, e.bits, e.off, e.seed_lo, e.seed_hi, e.words, e.mn, e.sc,
          nullptr, (int64_t)1, nullptr, nullptr, 0, e.short_len);
      return;
    }
  }
  quantize_pack_tile_body<DT, LPG_LOG2, B, false, false, false, tile_div<DT, LPG_LOG2>()>(
      static_cast<const u32x4*>(e.x), tile, wave_in_block, e.bits, e.off, e.seed_lo, e.seed_hi, e.words, e.mn, e.sc,
      nullptr, (int64_t)1, nullptr, nullptr);
}

template <int DT, int LPG_LOG2, bool METRICS, bool RELU>
hipError_t launch_tile(const daf_plan_t* p, const void* x, int64_t n_tiles, uint32_t seed_lo, uint32_t seed_hi,
                       uint32_t* out_words, float* out_min, float* out_scale, float* out_metrics, void* out_y,
                       hipStream_t stream) {
  using S = QTile<DT, LPG_LOG2>;
  const int short_len = (int)(p->n - n_tiles * S::kElems);            // elements after the whole tiles
#define DAF_LAUNCH(BITS)                                                                                   \
  do {                                                                                                     \
    auto kernel = k_quantize_pack_tile<DT, LPG_LOG2, BITS, false, METRICS, RELU, tile_div<DT, LPG_LOG2>()>; \
    const unsigned blocks = (unsigned)((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock) + (short_len > 0);   \
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), (tile_extra_lds<DT, LPG_LOG2, METRICS, RELU>(n_tiles)), \
                       stream, static_cast<const u32x4*>(x), n_tiles, p->d_bits, p->d_off, seed_lo, seed_hi,  \
                       out_words, out_min, out_scale,                                                      \
                       nullptr, (int64_t)1, out_metrics, static_cast<u32x4*>(out_y), short_len);           \
  } while (0)
  switch (p->uniform_bits) {
    case 0: DAF_LAUNCH(0); break;
    case 1: DAF_LAUNCH(1); break;
    case 2: DAF_LAUNCH(2); break;
    case 4: DAF_LAUNCH(4); break;
    case 8: DAF_LAUNCH(8); break;
    default: return hipErrorInvalidValue;
  }
#undef DAF_LAUNCH
  return hipGetLastError();
}

}  // namespace
