// The weight-gradient kernel for 16-bit formats and outputs of more than 256 rows: a
// tile of 512 (n) x 128 (k) on 8 waves, 32 values of m per step.  Included by unpack_matmul.hip, which
// holds the operand helpers, the tile order and the general kernel.
//
// What bounds it is the instructions next to the matrix ones: a step has 16 matrix instructions per wave (1024 cycles per
// SIMD with its two waves), and vector instructions, LDS reads and loads each showed up almost in full
// when they were left out.  Hence
//   - the tile is twice as wide in n as in earlier forms (256 x 256): a value of x is unpacked half as often,
//     8 instead of 16 codes per lane and step; grad_y, which needs no arithmetic, is fetched twice as often;
//   - grad_y goes from memory straight into LDS: no registers, no LDS stores by the waves;
//     (130 instead of 210 instructions per wave and step together);
//   - everything but the matrix instructions is dealt out to the slots behind them (do_step), operands are
//     read half a step ahead, so that a step begins and ends with matrix instructions whose operands are there
//     (the same instructions in the order they are thought of: 3.13 ms, dealt out: 2.97, on the 256 x 256 tile).
// 32768 x 4096 x 11008 bfloat16 {2,4,8}: 3.23 -> 2.65 ms (915 -> 1115 TFLOP/s; matrix cores busy 47 -> 67 % of
// the cycles, at 1.86 -> 1.59 GHz: the chip's power now sets the clock); 32768 x 3072 x 768 binary16 {1,2,4,8}: 213 ->
// 174 us.  Since then: 134 instead of 146 instructions per wave and step 2630 -> 2633 us (fewer cycles at a lower clock); 4 waves of 128 x 128
// with 512 registers each, a third less LDS traffic, 2908 (one wave per SIMD is bound by issue: 240 instructions in 1024 cycles).
#pragma once

namespace {

struct Wide {
  static constexpr int kBM = 32, kBN = 512, kBK = 128, kThreads = 512;
  // LDS, all of a compute unit's 160 KB.  Rows are unpadded (a load fills 1 KB of consecutive LDS) with the
  // 64-byte piece s of row r at place s ^ (r mod 4): the transposing reads take 64 bytes of four
  // consecutive rows at a time, which then lie on different banks.
  static constexpr int kGyRow = kBN * 2, kXRow = kBK * 2;
  static constexpr int kGyBytes = kBM * kGyRow, kXBytes = kBM * kXRow;
  static constexpr int kGyCopies = 4, kXCopies = 3;
  static constexpr int kRing = 4;                           // steps of group constants
  static constexpr int kGroupsPerRow = kBK / 32, kEntries = kBM * kGroupsPerRow;
  static constexpr int kXAt = kGyCopies * kGyBytes, kMetaAt = kXAt + kXCopies * kXBytes;
  static constexpr int kLdsBytes = kMetaAt + kRing * kEntries * 16;
  static_assert(kLdsBytes <= 160 * 1024, "LDS of a compute unit");
  static_assert(kEntries * 4 == kThreads, "a thread carries one of the four constants of one group");
};

// load_at for the loads that the wait at the end of a step counts: a relaxed atomic load (an ordinary load instruction
// at this scope) is never left out, doubled or moved past another load, whether its result is used or not.  Aligned.
__device__ __forceinline__ uint32_t counted_load(const void* uniform_base, uint32_t byte_off) {
  const char* base = static_cast<const char*>(uniform_base);
  return __hip_atomic_load(reinterpret_cast<const uint32_t*>(base + byte_off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

template <int DT, bool MIXED>
__global__ __launch_bounds__(Wide::kThreads, 2) void k_unpack_matmul_wide(
    const uint32_t* __restrict__ words, const float* __restrict__ mn, const float* __restrict__ scale,
    const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, uint32_t uniform_bits, int32_t gs,
    const void* __restrict__ grad_y, int64_t M, int64_t N, int64_t K, int32_t tiles_n, int32_t tiles_k,
    uint32_t whole, int32_t slices, float* __restrict__ out, float* __restrict__ partial) {
  using W = Wide;
  __shared__ __attribute__((aligned(1024))) char lds[W::kLdsBytes];

  const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
  const uint32_t uw = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave);
  const TileShare share = share_of(blockIdx.x, whole, slices, (uint32_t)tiles_n, (uint32_t)tiles_k, (int)(M / W::kBM));
  const int64_t n0 = (int64_t)share.tn * W::kBN, k0 = (int64_t)share.tk * W::kBK;
  const int steps = share.steps;
  const int64_t m_begin = (int64_t)share.first_step * W::kBM;
  // The last tile of n may reach past the output: its columns outside are read from column 0 instead and never stored.
  const uint32_t n_valid = (uint32_t)((N - n0) < W::kBN ? (N - n0) : W::kBN);

  // ---- grad_y: wave w loads rows 4 w .. 4 w + 3 of a step, one per instruction.
  const uint32_t row_bytes = (uint32_t)N * 2u;
  uint32_t gy_off[4];
#pragma unroll
  for (uint32_t r = 0; r < 4; ++r) {
    const uint32_t from = lane ^ (r << 2);                                // 16-byte pieces
    gy_off[r] = from * 8u < n_valid ? 16u * from : 0u;
  }
  const char* gy_src = uniform_pointer(reinterpret_cast<const char*>(grad_y) +
                                       ((m_begin + 4 * (int64_t)uw) * (int64_t)row_bytes + n0 * 2));
  const int64_t gy_stride = W::kBM * (int64_t)row_bytes;
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds);
  const uint32_t gy_dst = lds0 + uw * (4u * W::kGyRow);
  auto load_gy = [&](int q, int r) __attribute__((always_inline)) {       // q = 0, 1, 2, ...; past the end the last step again
    load_to_lds(gy_dst + (uint32_t)(q & (W::kGyCopies - 1)) * W::kGyBytes + (uint32_t)r * W::kGyRow, gy_off[r],
                gy_src + r * (int64_t)row_bytes);
    if (r == 3) gy_src += q + 1 < steps ? gy_stride : 0;
  };

  // ---- x: thread (co, xr) owns columns 8 co .. 8 co + 7 of row xr.
  const uint32_t co = t & 15u, xr = t >> 4;
  const uint32_t gpr = (uint32_t)(K / gs);                              // groups per row of x
  const uint32_t k_col = min((uint32_t)k0 + 8u * co, (uint32_t)K - 8u);   // (columns past the output: its last ones again, never stored)
  const uint32_t gk = k_col / (uint32_t)gs;
  const uint32_t in_group = k_col - gk * (uint32_t)gs;                  // a multiple of 8
  const uint32_t wpgb = (uint32_t)gs >> 5;                              // words per group and bit of width
  const uint32_t g_first = (uint32_t)k0 / (uint32_t)gs;
  const uint32_t n_groups = (min((uint32_t)k0 + (uint32_t)W::kBK, (uint32_t)K) - 1u) / (uint32_t)gs - g_first + 1u;
  const uint32_t my_entry = W::kMetaAt + 16u * (xr * (uint32_t)W::kGroupsPerRow + (gk - g_first));
  const uint32_t x_store = W::kXAt + xr * (uint32_t)W::kXRow + ((16u * co) ^ (64u * (xr & 3u)));

  // Group constants, {min, scale, word offset, width} per group: a thread carries one of the four of one group, which
  // one depends on its wave only.  No branch: the array is chosen by pointer.  A width is read with the aligned
  // word that holds it (a step's first group is a multiple of 32) and picked out when it is stored.  With one width for
  // all groups the upper four waves carry what the lower four do.
  const uint32_t field = MIXED ? uw >> 1 : (uw >> 1) & 1u;
  const uint32_t e = t & 127u, m_row = e / (uint32_t)W::kGroupsPerRow;
  const uint32_t m_j = min(e % (uint32_t)W::kGroupsPerRow, n_groups - 1u);   // (entries past the tile's groups hold the last one again)
  const uint32_t m_goff = m_row * gpr + g_first + m_j;                       // relative to the step's first group
  const bool is_width = field == 3u;
  const uint32_t skew = (uint32_t)reinterpret_cast<uintptr_t>(bits) & 3u;    // (the caller's array may start anywhere)
  const char* const meta_src = field == 0u   ? reinterpret_cast<const char*>(mn)
                               : field == 1u ? reinterpret_cast<const char*>(scale)
                               : field == 2u ? reinterpret_cast<const char*>(off)
                                             : reinterpret_cast<const char*>(bits) - skew;
  const int meta_log2 = is_width ? 0 : 2;
  const uint32_t meta_off = is_width ? (m_goff + skew) & ~3u : 4u * m_goff;
  const uint32_t meta_shift = is_width ? 8u * ((m_goff + skew) & 3u) : 0u, meta_mask = is_width ? 0xFFu : ~0u;
  const uint32_t meta_dst = W::kMetaAt + 16u * e + 4u * field;
  const int64_t g_begin = m_begin * (int64_t)gpr, g_stride = W::kBM * (int64_t)gpr;
  int64_t gu = g_begin;                                                      // first group of the step whose constants are requested next
  int meta_q = 0;
  auto meta_load = [&](uint32_t& v) __attribute__((always_inline)) {
    v = counted_load(meta_src + (gu << meta_log2), opaque(meta_off));
    gu += ++meta_q < steps ? g_stride : 0;
  };
  auto meta_store = [&](uint32_t v, int q) __attribute__((always_inline)) {
    *reinterpret_cast<uint32_t*>(lds + meta_dst + (uint32_t)(q & (W::kRing - 1)) * (W::kEntries * 16)) =
        MIXED ? (v >> meta_shift) & meta_mask : v;
  };
  struct Group { uint32_t off, b; };                                         // word offset and width of the thread's group in a step
  const uint32_t g_voff = xr * gpr + gk;
  auto fetch_group = [&](Group& g, int q) __attribute__((always_inline)) {
    if (MIXED) {
      const uint2 v = *reinterpret_cast<const uint2*>(lds + my_entry + (uint32_t)(q & (W::kRing - 1)) * (W::kEntries * 16) + 8);
      g.off = v.x;
      g.b = v.y;
    } else {
      const uint32_t i = (uint32_t)(g_begin + (int64_t)min(q, steps - 1) * g_stride) + g_voff;
      g.off = i * (wpgb * uniform_bits);
      g.b = uniform_bits;
    }
  };
  // The words of the thread's 8 codes: that of codes 0 .. 3 and that of codes 4 .. 7 (the next one with 8 bits, else the same).
  struct Codes { uint32_t wa, wb, b; };
  auto fetch_codes = [&](Codes& c, const Group& g) __attribute__((always_inline)) {
    const uint32_t w0 = g.off + (__umul24(in_group, g.b) >> 5);
    c.wa = counted_load(words, 4u * w0);
    c.wb = counted_load(words, 4u * (w0 + (g.b >> 3)));
    c.b = g.b;
  };
  auto read_scale = [&](int q) __attribute__((always_inline)) {              // {min, scale}
    return *reinterpret_cast<const float2*>(lds + my_entry + (uint32_t)(q & (W::kRing - 1)) * (W::kEntries * 16));
  };
  // Unpack, dequantize, round to the element format, store.  Element j of a group has its lowest bit at bit
  // -(j + 1) * b (mod 32) of its word; the extract takes its offset mod 32.
  struct Build { uint32_t wa, wb, b, sh; float v[8]; };
  auto begin_build = [&](Build& h, const Codes& c) __attribute__((always_inline)) {
    h.wa = c.wa;
    h.wb = c.wb;
    h.b = c.b;
    asm volatile("" : "+v"(h.wa), "+v"(h.wb));      // taken here: moved up over the barrier the unpacking would wait for newer loads
    h.sh = (uint32_t)__mul24((int)h.b, -(int)(in_group + 1u));
  };
  auto unpack_one = [&](Build& h, const float2& ms, int j) __attribute__((always_inline)) {
    h.v[j] = __builtin_fmaf((float)__builtin_amdgcn_ubfe(j < 4 ? h.wa : h.wb, h.sh, h.b), ms.y, ms.x);
    h.sh -= h.b;
  };
  auto end_build = [&](const Build& h, uint32_t x_copy) __attribute__((always_inline)) {
    *reinterpret_cast<uint4*>(lds + (x_store + x_copy)) =
        make_uint4(narrow16_pair<DT>(h.v[0], h.v[1]), narrow16_pair<DT>(h.v[2], h.v[3]),
                   narrow16_pair<DT>(h.v[4], h.v[5]), narrow16_pair<DT>(h.v[6], h.v[7]));
  };

  // ---- operands.  Lane l of 16-lane group G addresses row 8 (l / 32) + (l % 16) / 4 (plus 16 per half, plus 4 for the
  // second half of the operand) and the columns 16 (G % 2) + 4 (l % 4) .. of its 32-column block.
  const uint32_t li = lane & 31u, lg = lane >> 5;
  const uint32_t tr_row = 8u * lg + ((lane & 15u) >> 2), tr_col = 16u * ((lane >> 4) & 1u) + 4u * (lane & 3u);
  uint32_t a_read[2], b_read[4];
#pragma unroll
  for (uint32_t i = 0; i < 2; ++i) a_read[i] = tr_row * (uint32_t)W::kGyRow + (((2u * uw + i) ^ (tr_row & 3u)) << 6) + 2u * tr_col;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) b_read[j] = W::kXAt + tr_row * (uint32_t)W::kXRow + ((j ^ (tr_row & 3u)) << 6) + 2u * tr_col;
  struct Operands { uint4 a[2], b[4]; };
  auto read_operand = [&](Operands& o, uint32_t gy_copy, uint32_t x_copy, int half, int n) __attribute__((always_inline)) {   // n = 0 .. 5
    if (n < 2) o.a[n] = operand_tr(lds + (a_read[n] + gy_copy) + half * 16 * W::kGyRow, W::kGyRow);
    else o.b[n - 2] = operand_tr(lds + (b_read[n - 2] + x_copy) + half * 16 * W::kXRow, W::kXRow);
  };

  f32x16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  // ---- prologue, two trips to memory: the constants of steps 0 .. 9, then the words of steps 0 .. 4.  The constants of
  // steps 0 .. 5 go through the place of the grad_y copy that is loaded last (the ring has four slots).
  Codes codes[4];
  Group group;
  Operands op[2];
  uint32_t mv[4];
  float2 ms;
  constexpr uint32_t kFirst = 3 * W::kGyBytes - W::kMetaAt;     // from the ring to that place
  {
    uint32_t first[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) meta_load(first[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) meta_load(mv[q]);              // steps 6 to 9
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) load_gy(q, r);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const uint32_t v = MIXED ? (first[q] >> meta_shift) & meta_mask : first[q];
      *reinterpret_cast<uint32_t*>(lds + (meta_dst + kFirst) + q * (W::kEntries * 16)) = v;
      if (q >= 2) meta_store(first[q], q);
    }
    __syncthreads();
    Group g[6];
    float2 scales[3];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const uint4 c = *reinterpret_cast<const uint4*>(lds + (my_entry + kFirst) + q * (W::kEntries * 16));
      if (q < 3) scales[q] = make_float2(u2f(c.x), u2f(c.y));
      if (MIXED) {
        g[q].off = c.z;
        g[q].b = c.w;
      } else {
        fetch_group(g[q], q);
      }
    }
    Codes built[2];
    fetch_codes(built[0], g[0]);
    fetch_codes(built[1], g[1]);
#pragma unroll
    for (int q = 0; q < 3; ++q) fetch_codes(codes[q], g[q + 2]);
    codes[3] = codes[2];
    group = g[5];
    ms = scales[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      Build h;
      begin_build(h, built[q]);
#pragma unroll
      for (int j = 0; j < 8; ++j) unpack_one(h, scales[q], j);
      end_build(h, (uint32_t)(q * W::kXBytes));
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);               // the same, for the compiler's own counting
  __syncthreads();
#pragma unroll
  for (int n = 0; n < 6; ++n) read_operand(op[0], 0u, 0u, 0, n);

  // ---- step s: products of step s; step s + 2 of x is built; requested: grad_y of s + 3, words of s + 5, group
  // constants of s + 10.  Those of s + 6 enter the ring in the place of s + 2, whose minimum and scale are already in
  // registers; minimum and scale of s + 3 are read from it, and behind the barrier offset and width of s + 6.
  // LAST: one of the (at most three) steps after the last whole four: everything it needs has been requested, so it requests
  // nothing more and its wait counts nothing.
  uint32_t x_cur = 0u, x_next = W::kXBytes, x_build = 2 * W::kXBytes;
  auto do_step = [&](auto last, Codes& c, Codes& c_fill, Group& g, uint32_t& v, int s) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value != 0;
    const uint32_t gy_copy[2] = {(uint32_t)((s + 1) & (W::kGyCopies - 1)) * W::kGyBytes,      // [half that is read]
                                 (uint32_t)(s & (W::kGyCopies - 1)) * W::kGyBytes};
    const uint32_t x_copy[2] = {x_next, x_cur};
    Build h;
    float2 ms_next;
#pragma unroll
    for (int slot = 0; slot < 16; ++slot) {
      const int hs = slot >> 3, n = slot & 7;
      acc[n >> 2][n & 3] = mfma_32x32x16<DT>(op[hs].a[n >> 2], op[hs].b[n & 3], acc[n >> 2][n & 3]);
      if (n < 6) read_operand(op[hs ^ 1], gy_copy[hs ^ 1], x_copy[hs ^ 1], hs ^ 1, n);
      if (slot == 2) begin_build(h, c);
      if (slot >= 2 && slot < 10) {
        unpack_one(h, ms, slot - 2);
        asm volatile("" : "+v"(h.v[slot - 2]));     // here, not where it is stored
      }
      if (slot == 10) end_build(h, x_build);
      if (slot == 1) ms_next = read_scale(s + 3);
      if (!LAST && slot == 4) fetch_codes(c_fill, g);        // words of s + 5
      if (!LAST && slot == 6) {
        meta_store(v, s + 6);
        meta_load(v);                                        // constants of s + 10
      }
      if (!LAST && slot >= 11 && slot < 15) load_gy(s + 3, slot - 11);
      __builtin_amdgcn_sched_barrier(0);
    }
    // grad_y of s + 2 has landed when at most the loads behind it are in flight: two words and a constant of s, four
    // rows of grad_y of s + 3.  (All seven are loads that the compiler may not drop: counted_load, load_to_lds.)
    if (LAST)
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else
      asm volatile("s_waitcnt vmcnt(7) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (!LAST) fetch_group(g, s + 6);
    ms = ms_next;
    const uint32_t free_copy = x_cur;
    x_cur = x_next;
    x_next = x_build;
    x_build = free_copy;
  };
  int s = 0;
  for (; s + 4 <= steps; s += 4) {
    do_step(Index<0>{}, codes[0], codes[3], group, mv[0], s);
    do_step(Index<0>{}, codes[1], codes[0], group, mv[1], s + 1);
    do_step(Index<0>{}, codes[2], codes[1], group, mv[2], s + 2);
    do_step(Index<0>{}, codes[3], codes[2], group, mv[3], s + 3);
  }
  if (s < steps) do_step(Index<1>{}, codes[0], codes[3], group, mv[0], s);
  if (s + 1 < steps) do_step(Index<1>{}, codes[1], codes[0], group, mv[1], s + 1);
  if (s + 2 < steps) do_step(Index<1>{}, codes[2], codes[1], group, mv[2], s + 2);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may arrive in LDS after the work-group has ended

  // ---- epilogue: register r of a 32 x 32 block is row 8*(r/4) + 4*(lane/32) + r%4, column lane%32 ----
  if (64u * uw >= n_valid) return;
  float* dst = share.sliced ? partial + share.partial_tile * (int64_t)(W::kBN * W::kBK) : out + n0 * K + k0;
  const int64_t ld = share.sliced ? W::kBK : K;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (k0 + 32 * j >= K) break;                   // the last tile of k may reach 64 columns past the output
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t n = 64 * uw + 32 * i + 8 * (r >> 2) + 4 * lg + (r & 3);
        const int64_t k = 32 * j + li;
        dst[n * ld + k] = acc[i][j][r];
      }
    }
}

}  // namespace
