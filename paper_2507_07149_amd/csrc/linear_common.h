// Shared by the two kernels of the linear layer with a quantizing epilogue (linear_quantize.hip, linear_few_tiles.h): the matrix
// instruction, and the epilogue of one 32 x 32 block of the output.
#pragma once
#include "quantize_common.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <int DT>
__device__ __forceinline__ f32x16 mfma16(const u32x4& a, const u32x4& b, f32x16 c) {
  if constexpr (DT == kBF16) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
  }
}

// Two binary32 values rounded (nearest even) to the 16-bit format, low half first.
template <int DT>
__device__ __forceinline__ uint32_t round_pair(float lo, float hi) {
  if constexpr (DT == kBF16) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  } else {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    const f16x2 v = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, v);
  }
}

// The value held by the lane 32 away.
__device__ __forceinline__ uint32_t other_half(uint32_t v) {
  const u32x2 r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return (threadIdx.x & 32) ? r.x : r.y;
}
__device__ __forceinline__ float both_halves_min(float v) { return vmin(v, u2f(other_half(f2u(v)))); }
__device__ __forceinline__ float both_halves_max(float v) { return vmax(v, u2f(other_half(f2u(v)))); }

// Position -> output tile: panels of `panel` tile rows, column by column inside a panel (the last panel may be lower).
struct TileIndex {
  int m, n;
};
__host__ __device__ inline TileIndex tile_of_position(int pos, int tiles_m, int tiles_n, int panel_rows) {
  const int full = tiles_m / panel_rows * panel_rows;    // tile rows in whole panels
  TileIndex t;
  if (pos < full * tiles_n) {
    const int panel = pos / (panel_rows * tiles_n), in = pos % (panel_rows * tiles_n);
    t.m = panel * panel_rows + in % panel_rows;
    t.n = in / panel_rows;
  } else {
    const int rows = tiles_m - full, in = pos - full * tiles_n;
    t.m = full + in % rows;
    t.n = in / rows;
  }
  return t;
}

// ---- epilogue of one block.  Register r of a 32 x 32 block: n = 8*(r/4) + 4*(lane/32) + r%4, m = lane%32. ----
// The block rounded to the format: this lane's 16 consecutive n of row m, from 16 * (lane / 32) on, two to a dword.
template <int DT>
__device__ __forceinline__ void block_row(const f32x16& acc, uint32_t (&yv)[8]) {
  uint32_t d[4][2];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    d[j][0] = round_pair<DT>(acc[4 * j], acc[4 * j + 1]);
    d[j][1] = round_pair<DT>(acc[4 * j + 2], acc[4 * j + 3]);
  }
  // Lower half-wave: runs j = 0..3 are n 0-3, 8-11, 16-19, 24-27; upper: 4-7, 12-15, 20-23, 28-31.
  // Swapping the upper half of run 0 with the lower half of run 2 (and 1 with 3) leaves n 0-15
  // in the lower half-wave and n 16-31 in the upper one.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const u32x2 r02 = __builtin_amdgcn_permlane32_swap(d[0][h], d[2][h], false, false);
    const u32x2 r13 = __builtin_amdgcn_permlane32_swap(d[1][h], d[3][h], false, false);
    yv[h] = r02.x;
    yv[2 + h] = r02.y;
    yv[4 + h] = r13.x;
    yv[6 + h] = r13.y;
  }
}

// Widens it, and this lane's minimum and maximum.
template <int DT>
__device__ __forceinline__ void widen_row(const uint32_t (&yv)[8], float (&xf)[16], float& mn, float& mx) {
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const uint32_t pair = yv[e >> 1];
    xf[e] = DT == kBF16 ? u2f((e & 1) ? (pair & 0xFFFF0000u) : (pair << 16))
                        : widen16<DT>((e & 1) ? (pair >> 16) : (pair & 0xFFFFu));
  }
  mn = vmin(xf[0], xf[1]);
  mx = vmax(xf[0], xf[1]);
#pragma unroll
  for (int e = 2; e < 16; e += 2) {
    mn = vmin3(mn, xf[e], xf[e + 1]);
    mx = vmax3(mx, xf[e], xf[e + 1]);
  }
}

// A group as the element map needs it.
struct LinearGroup {
  float mn, inv, invs;
  uint32_t b;
  bool any_exact2;                     // of the wave: rare, the whole wave branches
  uint32_t* words;                     // the group's first word
};
__device__ __forceinline__ LinearGroup linear_group(const GroupScale& gs, uint32_t b, uint32_t* words) {
  LinearGroup g;
  g.mn = gs.mn;
  g.inv = gs.inv;
  g.invs = gs.inv * kScale;
  g.b = b;
  g.any_exact2 = __builtin_amdgcn_ballot_w64(!(g.invs <= 3.402823466e+38f)) != 0ull;   // 256 is then applied to the rounded product
  g.words = words;
  return g;
}

// Widths and offsets of GROUPS (1, 2 or 4) consecutive groups of a row, the first one's number a multiple of GROUPS, from the plan's own
// copies, which begin at multiples of 16 bytes.
template <int GROUPS>
struct RowGroups {
  struct alignas(GROUPS) { uint8_t of[GROUPS]; } b;
  struct alignas(4 * GROUPS) { uint32_t of[GROUPS]; } off;
};
template <int GROUPS>
__device__ __forceinline__ RowGroups<GROUPS> row_groups(const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, int64_t g) {
  RowGroups<GROUPS> r;
  r.b = *reinterpret_cast<const decltype(r.b)*>(bits + g);
  r.off = *reinterpret_cast<const decltype(r.off)*>(off + g);
  return r;
}

// Quantizes and packs the lane's 16 elements; `e0` is the first one's place in the group, `flat` in the tensor.
__device__ __forceinline__ void quantize_row(const float (&xf)[16], const LinearGroup& g, uint32_t e0, int64_t flat,
                                             uint32_t seed_lo, uint32_t seed_hi, int lg) {
  const uint4 rnd4 = philox_block<true>((uint64_t)(flat >> 4), seed_lo, seed_hi);
  const uint32_t b = g.b;
  uint32_t q[4];                                           // four codes each, first element in the most significant byte
  auto codes = [&](auto two_products, float mult) {
#pragma unroll
    for (int c = 0; c < 4; c += 2) {
      int t[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) t[e] = neg_position<decltype(two_products)::value>(g.mn - xf[4 * c + e], mult);
      code_bytes(t, c ? rnd4.z : rnd4.x, c ? rnd4.w : rnd4.y, q[c], q[c + 1]);
    }
  };
  if (g.any_exact2) {
    // lanes that do not need it multiply by 256 afterwards too: a power of two, the same product
    codes(std::true_type{}, g.inv);
  } else {
    codes(std::false_type{}, g.invs);
  }
  uint32_t* dst = g.words;
  if (b == 8u) {
    typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(4)));
    *reinterpret_cast<u32x4_any*>(dst + (e0 >> 2)) = u32x4_any{q[0], q[1], q[2], q[3]};
  } else if (b == 4u) {
    dst[(e0 >> 3)] = pack_codes<4>(q[0], q[1]);
    dst[(e0 >> 3) + 1] = pack_codes<4>(q[2], q[3]);
  } else if (b == 2u) {
    dst[e0 >> 4] = (pack_codes<2>(q[0], q[1]) << 16) | pack_codes<2>(q[2], q[3]);
  } else {
    const uint32_t half = (pack_codes<1>(q[0], q[1]) << 8) | pack_codes<1>(q[2], q[3]);
    const uint32_t upper = other_half(half);               // the lane 32 away runs the same branch: same group, same width
    if (lg == 0) dst[e0 >> 5] = (half << 16) | upper;
  }
}

}  // namespace
