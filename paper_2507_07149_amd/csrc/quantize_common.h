// Shared by the quantize kernels of every route: launch shape, Eq. 1 per group (scale and the
// reciprocal used by the element map), the negated element map itself, the fused max(z, 0).
// Included by quantize_pack.hip only (once per element format).
#pragma once
#include <type_traits>

#include "daf_device.h"
#include "daf_internal.h"

namespace {

using namespace daf;

constexpr int kWavesPerBlock = 4;
constexpr int kThreads = kWave * kWavesPerBlock;
constexpr float kScale = 256.0f;            // 2^kRandBits
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct GroupScale {
  float mn, scale, inv;
};

// Eq. 1 (left) per group, plus the reciprocal used for the per-element map.
__device__ __forceinline__ GroupScale group_scale(float mn, float mx, uint32_t b) {
  GroupScale s;
  s.mn = mn + 0.0f;                               // a zero minimum is stored as +0
  const float mxc = mx + 0.0f;
  const float L = (float)((1u << b) - 1u);
  const float range = mxc - s.mn;
  s.scale = range / L;
  float inv = 0.0f;
  if (range > 0.0f) {
    inv = L / range;
    if (!(inv <= 3.402823466e+38f)) inv = 0.0f;   // reciprocal overflowed
  }
  s.inv = inv;
  return s;
}

// What the element map rounds: -(256*floor(v) + T), with v the element's position on its group's grid and T the number of
// byte values for which it rounds up.  EXACT2 = false: invs = inv*256 (finite).  EXACT2 = true: invs = inv, and the
// factor 256 is applied to the rounded product.
template <bool EXACT2>
__device__ __forceinline__ int neg_position(float d, float invs) {   // d = mn - x
  float w = d * invs;
  if (EXACT2) w = w * kScale;
  return round_half_up_to_int(w);
}

// Negated code of one element.
template <bool EXACT2>
__device__ __forceinline__ int neg_code(float x, float mn, float invs, uint32_t r, int* t_out = nullptr) {
  const int t = neg_position<EXACT2>(mn - x, invs);
  if (t_out) *t_out = t;
  return (t + (int)r) >> 8;
}

// The codes of four (eight) consecutive elements, one to a byte, the first in the most significant one.  t: neg_position;
// not_rnd: the complement of their random bytes, element e's in byte e.  With r a byte and r' = 255 - r its complement,
// code = -((t + r) >> 8) = (r' - t) >> 8, which is byte 1 of the 16-bit value r' - t (t >= -255 * 256): two such values go to
// the halves of one register by the instruction that subtracts them anyway, and a byte permutation brings four codes
// together.  Shifting each out and into an accumulator took two instructions per element.  With the bytes packed by dot products
// and stored without branches (store_by_width) a binary16 tile of 4096 elements with four widths takes 784 vector instructions
// a wave instead of 956: 25 M elements both directions 27.0 -> 26.0 us, rows of 768 and 3072 73.2 -> 70.4, 361 M
// bfloat16 elements with metrics, selection and plan 280.5 -> 268.9.  (A register that
// an instruction has written in part is read two instructions later at the earliest: one wait state.)
#define DAF_HALF(OUT, HALF, KEEP, RND, BYTE, T) \
  "v_sub_u32_sdwa " OUT ", " RND ", " T " dst_sel:WORD_" HALF " dst_unused:UNUSED_" KEEP " src0_sel:BYTE_" BYTE " src1_sel:DWORD\n"
__device__ __forceinline__ uint32_t code_bytes(const int (&t)[4], uint32_t not_rnd) {
  uint32_t q, p;
  asm(DAF_HALF("%0", "0", "PAD", "%2", "1", "%4") DAF_HALF("%1", "0", "PAD", "%2", "3", "%6")
      DAF_HALF("%0", "1", "PRESERVE", "%2", "0", "%3") DAF_HALF("%1", "1", "PRESERVE", "%2", "2", "%5")
      "s_nop 0\n"
      "v_perm_b32 %0, %0, %1, %7\n"
      : "=&v"(q), "=&v"(p)
      : "v"(not_rnd), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "s"(0x07050301u));
  return q;
}
__device__ __forceinline__ void code_bytes(const int (&t)[8], uint32_t not_rnd0, uint32_t not_rnd1, uint32_t& q0, uint32_t& q1) {
  uint32_t p0, p1;
  asm(DAF_HALF("%0", "0", "PAD", "%4", "1", "%7") DAF_HALF("%2", "0", "PAD", "%4", "3", "%9")
      DAF_HALF("%1", "0", "PAD", "%5", "1", "%11") DAF_HALF("%3", "0", "PAD", "%5", "3", "%13")
      DAF_HALF("%0", "1", "PRESERVE", "%4", "0", "%6") DAF_HALF("%2", "1", "PRESERVE", "%4", "2", "%8")
      DAF_HALF("%1", "1", "PRESERVE", "%5", "0", "%10") DAF_HALF("%3", "1", "PRESERVE", "%5", "2", "%12")
      "v_perm_b32 %0, %0, %2, %14\n"
      "v_perm_b32 %1, %1, %3, %14\n"
      : "=&v"(q0), "=&v"(q1), "=&v"(p0), "=&v"(p1)
      : "v"(not_rnd0), "v"(not_rnd1), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3]), "v"(t[4]), "v"(t[5]), "v"(t[6]), "v"(t[7]),
        "s"(0x07050301u));
}
#undef DAF_HALF

// Four code bytes as bits, first code most significant: by a dot product with the powers of the width, whose weights are
// bytes too (1 and 2 bits), or in two steps (4 bits, whose byte pairs are joined first).
__device__ __forceinline__ uint32_t dot_bytes(uint32_t a, uint32_t weights, uint32_t c) {
  return __builtin_amdgcn_udot4(a, weights, c, false);
}
constexpr uint32_t kWeights1 = 0x08040201u, kWeights1Upper = 0x80402010u, kWeights2 = 0x40100401u;
// Bytes 2 and 0 of the result are the joined pairs of 4-bit codes; the others are of no use.
__device__ __forceinline__ uint32_t join_pairs4(uint32_t q) { return q | (q >> 4); }
// Four (eight) code bytes of B = 1, 2 or 4 bits; above the 4 B (8 B) bits other bits may stand.
template <int B>
__device__ __forceinline__ uint32_t pack_codes(uint32_t q) {
  if (B == 4) {
    const uint32_t j = join_pairs4(q);
    return __builtin_amdgcn_perm(j, j, 0x0C0C0200u);
  }
  return dot_bytes(q, B == 2 ? kWeights2 : kWeights1, 0u);
}
template <int B>
__device__ __forceinline__ uint32_t pack_codes(uint32_t q0, uint32_t q1) {
  if (B == 4) return __builtin_amdgcn_perm(join_pairs4(q0), join_pairs4(q1), 0x06040200u);
  if (B == 2) return dot_bytes(q1, kWeights2, dot_bytes(q0, kWeights2, 0u) << 8);
  return dot_bytes(q1, kWeights1, dot_bytes(q0, kWeights1Upper, 0u));
}

// T * (256 - T) for the element whose rounded product is t: 65536 * p * (1 - p) with p = T / 256
// the probability of rounding up (T = 256, always up, reads as 0 here: the same product).
__device__ __forceinline__ uint32_t sr_variance_term(int t) {
  const uint32_t T = (uint32_t)(-t) & 255u;
  return T * (256u - T);
}

// The sum of sr_variance_term over four elements, as 256 * sum(T) - sum(T^2): the low bytes of the four t are
// brought together and two dot products do the rest, 5 instructions instead of 16.  (The term is the same for
// T and 256 - T, so the byte of t itself will do, and 0 stands for 256.)  The metrics variant of the tile kernel is
// bound by vector instructions alone; with this and sums over the lanes two loads at a time it takes 25
// per bfloat16 element instead of 28: 360 M elements, groups of 64, 245 -> 233 us, 90 M binary32 elements 116 -> 103 us.
__device__ __forceinline__ void sr_variance_sums(const int (&t)[4], uint32_t& sum, uint32_t& sum_sq) {
  const uint32_t lo = __builtin_amdgcn_perm((uint32_t)t[1], (uint32_t)t[0], 0x0C0C0400u);
  const uint32_t hi = __builtin_amdgcn_perm((uint32_t)t[3], (uint32_t)t[2], 0x04000C0Cu);
  const uint32_t bytes = lo | hi;
  sum = __builtin_amdgcn_udot4(bytes, 0x01010101u, sum, false);
  sum_sq = __builtin_amdgcn_udot4(bytes, bytes, sum_sq, false);
}

// max(x, +0) on the raw bits of one 32-bit word (one binary32 value or two 16-bit values):
// a value whose sign bit is set (negative, or -0) is a negative integer and becomes +0, any
// other value is kept; for finite inputs that is x > 0 ? x : +0 exactly.
template <int DT>
__device__ __forceinline__ uint32_t relu_bits(uint32_t w) {
  if (DT == kF32) {
    const int32_t v = (int32_t)w;
    return (uint32_t)(v > 0 ? v : 0);
  }
  typedef short short2v __attribute__((ext_vector_type(2)));
  const short2v v = __builtin_bit_cast(short2v, w);
  const short2v zero = {0, 0};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, zero));
}

}  // namespace
