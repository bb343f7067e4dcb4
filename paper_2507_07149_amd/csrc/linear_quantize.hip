// Producer fusion into a matrix product: y = x W^T of a linear layer, with the quantize+pack of y
// (Sec. 2.2 Eq. 1, Sec. 3.3) as the epilogue of the output tile, so that the activation the
// next layer saves is reduced, quantized and packed inside the kernel that produces it
// (Sec. 3.2.3) and is never read back from memory for that purpose.
//
//   x [M, K], W [N, K], y [M, N], all in one 16-bit format, row-major; products accumulated in
//   binary32 on the matrix cores (v_mfma_f32_32x32x16_bf16 / _f16), y rounded to the format with
//   round-to-nearest-even.  Groups are runs of 32, 64 or 128 consecutive elements of a row of y
//   (the flat grouping of daf_plan with such a group size, N being a multiple of 256), so a
//   group lies inside one wave's 64 x 128 part of the 256 x 256 output tile.
//
// The product is computed transposed (W supplies the rows of each 32 x 32 block, x the columns):
// a lane then holds, for ONE row m of y, four runs of four consecutive n per block, and after
// two half-wave swaps 16 consecutive n: one Philox block, 32 contiguous bytes of y, a whole
// number of packed words for every width but 1 (where the two lanes of a row put their halves
// together).  Minimum and maximum of a group are then a reduction inside a lane plus one
// exchange with the lane 32 away.  The element map, the random bytes and the word layout are
// those of daf_quantize_pack, so words, min and scale equal daf_quantize_pack(y) bit for bit.
#include "linear_few_tiles.h"

namespace {

constexpr int kLinThreads = 512;             // 8 waves: 4 along m x 2 along n
constexpr int kBM = 256, kBN = 256, kBK = 64;
constexpr int kRowBytes = kBK * 2;           // bytes of a staged row: one cache line
constexpr int kOperandBytes = 256 * kRowBytes;

// blockIdx -> tile.  Whole rounds of 256 workgroups: the s-th workgroup of die d in round r takes
// position 256 r + 32 d + s; the rest keep their index.  A bijection, as tile_of_position is.
__host__ __device__ inline TileIndex tile_of_workgroup(int id, int tiles_m, int tiles_n) {
  constexpr int kDies = 8, kPerDie = 32, kPanel = 4;
  const int total = tiles_m * tiles_n;
  int pos = id;
  if (id < total / (kDies * kPerDie) * (kDies * kPerDie)) {
    const int die = id % kDies, seq = id / kDies;
    pos = (seq / kPerDie) * (kDies * kPerDie) + die * kPerDie + seq % kPerDie;
  }
  return tile_of_position(pos, tiles_m, tiles_n, kPanel);
}

// Main loop.  The product is bound by feeding the compute units: 64 KB of operands per workgroup and step
// of 64 k, against 2048 cycles of matrix instructions.  What was measured on 32768 x 11008 x 4096 (the
// product alone, bfloat16; the chip holds about 1.6 GHz under this load):
//   1105 TFLOP/s  tiles loaded into registers, written to LDS a step later, one barrier per step
//   1200          loads straight into LDS, ring of four slots of 32 k (rows of 64 bytes)
//   1230          the same, the loads spread between the matrix instructions (issued in one run behind
//                 the barrier they hold up the wave while the matrix cores idle)
//   1340          rows of 128 bytes, whole cache lines, instead of 64
//   1500          without any loads in the loop (results meaningless: the ceiling of this structure)
// A step's tile is consumed in four phases, one per 32 rows of W (part nb), and x's rows belong to two parts
// (mb).  The operands of a phase are read from LDS one phase ahead, x's one step ahead, so that a part of a
// copy is free again long before its step has ended and the next loads into it start 2 to 3 halves
// before they are waited for:
//   half 0 (parts 0, 1) reads W1 W2 of s, x0 of s + 1;  loads x1 W0 of s + 2, W3 of s + 1
//   half 1 (parts 2, 3) reads W3 of s, W0 x1 of s + 1;  loads W1 W2 of s + 2, x0 of s + 3
// Every part is overwritten only in a half after the one that read it (the barrier between the halves follows a
// wait for the reads), and is read only after the barrier behind "all but the last eight loads have
// landed": the loads of two halves stay in flight, four per wave and half.
//
// Rows of 128 bytes are stored unpadded (a load writes 1 KB of consecutive LDS) with the 16-byte piece p
// of row r at place p ^ (r / 2 mod 8): no bank conflicts in the counters.

template <int DT, int GS_LOG2, bool MIXED, bool QUANT>
__global__ __launch_bounds__(kLinThreads, 2) void k_linear_quantize_pack(
    const char* __restrict__ x, const char* __restrict__ w, int M, int N, int K, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t uniform_b, const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, char* __restrict__ y,
    uint32_t* __restrict__ words, float* __restrict__ out_min, float* __restrict__ out_scale) {
  __shared__ __align__(1024) char lds[4 * kOperandBytes];      // W of even and odd steps, x of even and odd steps
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t >> 6;
  const int wm = wave & 3, wn = wave >> 2;
  const int li = lane & 31, lg = lane >> 5;

  // Workgroups are handed to the eight dies in turn, so the 32 workgroups that run together on one
  // die (32 compute units, one cache) are every eighth one.  They get 32 consecutive positions
  // of an order that walks panels of four tile rows column by column: a patch of about 4 x 8
  // tiles, whose workgroups, moving through k in step, share four slabs of x and eight of W in
  // that cache instead of one and thirty-two.
  const int tiles_n = N / kBN, tiles_m = M / kBM;
  const TileIndex ti = tile_of_workgroup((int)blockIdx.x, tiles_m, tiles_n);
  const int tm = ti.m, tn = ti.n;
  const int64_t m0 = (int64_t)tm * kBM, n0 = (int64_t)tn * kBN;

  f32x16 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  const int steps = K / kBK;
  const int64_t row_bytes = (int64_t)K * 2;
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds);
  const int uw = __builtin_amdgcn_readfirstlane(wave);

  // What a wave loads: of part nb of W (rows 32 nb ... of either half) eight rows, of part mb of x
  // (rows 32 mb ... of each quarter) two times eight.
  const int w_row = (uw >> 2) * 128 + (uw & 3) * 8, x_row = (uw >> 1) * 64 + (uw & 1) * 16;
  const int l_row = lane >> 3;
  const uint32_t l_off = (uint32_t)(l_row * row_bytes);
  const uint32_t piece = (uint32_t)((lane & 7) ^ (l_row >> 1));          // rows 0..7 of sixteen
  const uint32_t off_even = l_off + (piece << 4), off_odd = l_off + ((piece ^ 4u) << 4);
  const uint32_t off_w = (uw & 1) ? off_odd : off_even;
  const char *src_w[4], *src_x[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i) src_w[i] = uniform_pointer(w + (n0 + w_row + 32 * i) * row_bytes);
#pragma unroll
  for (int i = 0; i < 4; ++i) src_x[i >> 1][i & 1] = uniform_pointer(x + (m0 + x_row + 32 * (i >> 1) + 8 * (i & 1)) * row_bytes);
  const uint32_t dst_w = lds0 + (uint32_t)w_row * kRowBytes, dst_x = lds0 + 2 * kOperandBytes + (uint32_t)x_row * kRowBytes;
  // Part nb of W of step `s`.  Past the end the last step again (never used): the loop has no branches around loads.
  auto fetch_w = [&](int nb, int s) {
    load_to_lds(dst_w + (uint32_t)((s & 1) * kOperandBytes + nb * 32 * kRowBytes), off_w, src_w[nb]);
    src_w[nb] += s + 1 < steps ? kRowBytes : 0;
  };
  auto fetch_x = [&](int mb, int j, int s) {
    load_to_lds(dst_x + (uint32_t)((s & 1) * kOperandBytes + (mb * 32 + j * 8) * kRowBytes), j ? off_odd : off_even,
                src_x[mb][j]);
    src_x[mb][j] += s + 1 < steps ? kRowBytes : 0;
  };

  // Operand reads: lane li of a block reads the 16-byte piece 2 ks + lg of row li, found at piece ^ (row / 2 mod 8).
  const char *pa[4], *pb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int col = ((2 * ks + lg) ^ ((li >> 1) & 7)) << 4;
    pa[ks] = lds + (wn * 128 + li) * kRowBytes + col;
    pb[ks] = lds + 2 * kOperandBytes + (wm * 64 + li) * kRowBytes + col;
  }
  auto read_a = [&](int nb, int ks, int parity) {
    return *reinterpret_cast<const u32x4*>(pa[ks] + parity * kOperandBytes + nb * 32 * kRowBytes);
  };
  auto read_b = [&](int mb, int ks, int parity) {
    return *reinterpret_cast<const u32x4*>(pb[ks] + parity * kOperandBytes + mb * 32 * kRowBytes);
  };

  u32x4 a[2][4], b[2][2][4];                 // a[nb % 2][ks], b[step % 2][mb][ks]
  fetch_x(0, 0, 0); fetch_x(0, 1, 0); fetch_x(1, 0, 0); fetch_x(1, 1, 0); fetch_w(0, 0);
  fetch_w(1, 0); fetch_w(2, 0); fetch_x(0, 0, 1); fetch_x(0, 1, 1);
  fetch_x(1, 0, 1); fetch_x(1, 1, 1); fetch_w(0, 1); fetch_w(3, 0);
  asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    b[0][0][ks] = read_b(0, ks, 0);
    b[0][1][ks] = read_b(1, ks, 0);
    a[0][ks] = read_a(0, ks, 0);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  fetch_w(1, 1); fetch_w(2, 1); fetch_x(0, 0, 2); fetch_x(0, 1, 2);
  asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // One step on the copies of parity P; two halves of sixteen matrix instructions, a barrier behind each.
  auto step = [&](auto parity, int s) {
    constexpr int P = decltype(parity)::value;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {                              // k pieces 2h and 2h + 1 of part nb
        acc[0][nb] = mfma16<DT>(a[nb & 1][2 * h], b[P][0][2 * h], acc[0][nb]);
        __builtin_amdgcn_sched_barrier(0);
        if (nb == 0) fetch_x(1, h, s + 2);
        else if (nb == 1) { if (h == 0) fetch_w(0, s + 2); else fetch_w(3, s + 1); }
        else if (nb == 2) fetch_w(1 + h, s + 2);
        else fetch_x(0, h, s + 3);
        __builtin_amdgcn_sched_barrier(0);
        a[(nb + 1) & 1][2 * h] = nb < 3 ? read_a(nb + 1, 2 * h, P) : read_a(0, 2 * h, P ^ 1);
        a[(nb + 1) & 1][2 * h + 1] = nb < 3 ? read_a(nb + 1, 2 * h + 1, P) : read_a(0, 2 * h + 1, P ^ 1);
        b[P ^ 1][nb >> 1][2 * (nb & 1) + h] = read_b(nb >> 1, 2 * (nb & 1) + h, P ^ 1);
        acc[1][nb] = mfma16<DT>(a[nb & 1][2 * h], b[P][1][2 * h], acc[1][nb]);
        acc[0][nb] = mfma16<DT>(a[nb & 1][2 * h + 1], b[P][0][2 * h + 1], acc[0][nb]);
        acc[1][nb] = mfma16<DT>(a[nb & 1][2 * h + 1], b[P][1][2 * h + 1], acc[1][nb]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (nb & 1) {
        asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
    }
  };
  int s = 0;
  for (; s + 1 < steps; s += 2) {
    step(std::integral_constant<int, 0>{}, s);
    step(std::integral_constant<int, 1>{}, s + 1);
  }
  if (s < steps) step(std::integral_constant<int, 0>{}, s);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // ---- epilogue, by blocks of 32 x 32 (linear_common.h) ----
  // Widths and offsets of the lane's groups, one load each for those of a row, behind the last operands and before the stores of y: after
  // those every wait for one of them was a wait for the stores as well (loads and stores are counted together, in order), four
  // times a tile; in front of the first operands they hold those up.  bfloat16, {2,4,8}, group by group where they are used / one load a row in
  // front of the first operands / here: groups of 32 8960 x 1024 x 512 25.3 / 23.3 / 23.4 us, 8192 x 4096 x 512 62.1 / 61.3 / 60.4, 32768 x 2048 x 512
  // 116.7 / 114.0 / 113.0; of 64 8192 x 4096 x 512 56.4 / 55.4 / 55.2, 32768 x 768 x 3072 142 / 138 / 139; of 128 8192 x 4096 x 512
  // 52.9 / 53.7 / 53.1, 8192 x 11008 x 256 115.1 / 115.2 / 113.0.
  constexpr int kGs = 1 << GS_LOG2, kBlocksPerGroup = kGs / 32, kGroups = 4 / kBlocksPerGroup;
  [[maybe_unused]] RowGroups<kGroups> row[2];
  if constexpr (QUANT && MIXED) {
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
      row[mb] = row_groups<kGroups>(bits, off, ((m0 + wm * 64 + mb * 32 + li) * N + n0 + wn * 128) >> GS_LOG2);
    asm volatile("" ::: "memory");
  }
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) {
    const int64_t m = m0 + wm * 64 + mb * 32 + li;
    const int64_t n_lane = n0 + wn * 128 + lg * 16;             // + 32 nb: this lane's 16 consecutive n of block nb
    float xf[4][16];
    float bmn[4], bmx[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      uint32_t yv[8];
      block_row<DT>(acc[mb][nb], yv);
      char* dst = y + (m * N + n_lane + nb * 32) * 2;
      *reinterpret_cast<u32x4*>(dst) = u32x4{yv[0], yv[1], yv[2], yv[3]};
      *reinterpret_cast<u32x4*>(dst + 16) = u32x4{yv[4], yv[5], yv[6], yv[7]};
      widen_row<DT>(yv, xf[nb], bmn[nb], bmx[nb]);
    }
    if (!QUANT) continue;                                        // the product alone
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      float mn = bmn[gi * kBlocksPerGroup], mx = bmx[gi * kBlocksPerGroup];
#pragma unroll
      for (int q = 1; q < kBlocksPerGroup; ++q) {
        mn = vmin(mn, bmn[gi * kBlocksPerGroup + q]);
        mx = vmax(mx, bmx[gi * kBlocksPerGroup + q]);
      }
      mn = both_halves_min(mn);
      mx = both_halves_max(mx);
      const int64_t g = (m * N + n0 + wn * 128 + gi * kGs) >> GS_LOG2;
      const uint32_t b = MIXED ? (uint32_t)row[mb].b.of[gi] : uniform_b;
      const uint32_t woff = MIXED ? row[mb].off.of[gi] : (uint32_t)(g * (int64_t)((kGs * uniform_b) >> 5));
      const GroupScale gs = group_scale(mn, mx, b);
      if (lg == 0) {
        out_min[g] = gs.mn;
        out_scale[g] = gs.scale;
      }
      const LinearGroup group = linear_group(gs, b, words + woff);
#pragma unroll
      for (int q = 0; q < kBlocksPerGroup; ++q) {
        const int nb = gi * kBlocksPerGroup + q;
        quantize_row(xf[nb], group, (uint32_t)(q * 32 + lg * 16), m * N + n_lane + nb * 32, seed_lo, seed_hi, lg);
      }
    }
  }
}

// How an output is tiled: the first `whole` 256 x 256 tiles of the sequence as they are, whole rounds of 256 workgroups
// (k_linear_quantize_pack), the rest cut into `cut` each (1: not cut, in the same launch; 2, 4, 8, 16: k_linear_few_tiles).
// The estimate: a round of 256 workgroups takes `fixed` (first operands, epilogue, last waves) and `step` per 64 values of k, each
// between its value for a lone workgroup and for a full chip (shared cache and memory, clock).  Microseconds, fitted to
// 23 shapes of 1 to 768 tiles of 256 x 256 and K = 256, 1024, 4096, all five forms measured on each; the form picked was
// 0.7 % behind the best on average, 10 % at most.  Some of them, whole call, bfloat16, {2,4,8} or 4 bits:
//   tiles of 256 x 256, K    1      2      4      8     16
//       1, 1024           24.7   16.3    9.9    8.4    8.5
//      16, 4096           67.9   39.9   25.1   19.4   17.5
//      64, 1024           28.1   19.3   15.3   18.8   25.9
//     100, 1024           27.9   21.9   24.4   32.0   37.2
//     128, 4096           74.2   61.5   70.8   91.2  132.8
//     192, 1024           34.3   43.7   43.8   52.3   66.4
//     300, 4096          179.4  168.2  179.0  225.3  327.2
struct LinearTiling {
  int64_t whole;
  int cut;
};
LinearTiling linear_tiling(int64_t M, int64_t N, int64_t K) {
  static constexpr struct {
    int cut;
    float fixed_lone, fixed_full, step_lone, step_full;
  } kForms[] = {{1, 7.9f, 12.6f, 0.82f, 1.38f}, {2, 6.3f, 9.2f, 0.41f, 0.78f}, {4, 1.9f, 4.9f, 0.26f, 0.48f},
                {8, 0.0f, 3.3f, 0.21f, 0.29f},  {16, 2.5f, 2.4f, 0.11f, 0.19f}};
  const float steps = (float)(K / kBK);
  auto estimate = [&](int form, int64_t tiles) {
    const auto& f = kForms[form];
    const int64_t rounds = tiles * f.cut / 256, rest = tiles * f.cut % 256;
    const float busy = (float)rest / 256.0f;
    float time = (float)rounds * (f.fixed_full + steps * f.step_full);
    if (rest > 0)
      time += f.fixed_lone + busy * (f.fixed_full - f.fixed_lone) + steps * (f.step_lone + busy * (f.step_full - f.step_lone));
    return time;
  };
  constexpr float kSecondLaunch = 4.0f;            // the gap between the two; with the rest cut, bfloat16, groups of 64, before and now:
                                                   // 272 tiles, K 1024 65.7 / 49.2 us, 300, 4096 189 / 156, 576, 1024 117 / 107, 1056, 2048 306 / 286
  const int64_t tiles = (M / kBM) * (N / kBN), rounds = tiles / 256 * 256;
  LinearTiling best = {tiles, 1};
  float best_time = estimate(0, rounds) + 0.97f * estimate(0, tiles - rounds);   // at equal estimates the form that moves the fewest bytes
  for (int form = 1; form < 5; ++form)
    for (const int64_t whole : {(int64_t)0, rounds}) {
      if (whole == tiles || (whole == 0 && rounds > 256)) continue;
      const float time = estimate(0, whole) + estimate(form, tiles - whole) + (whole > 0 ? kSecondLaunch : 0.0f);
      if (time < best_time) {
        best = {whole, kForms[form].cut};
        best_time = time;
      }
    }
  return best;
}

template <int DT, int GS_LOG2>
hipError_t launch_gs(const daf_plan_t* p, const void* x, const void* w, int M, int N, int K, uint64_t seed, void* y,
                     uint32_t* words, float* mn, float* sc, hipStream_t stream) {
  const uint32_t lo = (uint32_t)seed, hi = (uint32_t)(seed >> 32);
  const bool quant = words != nullptr, mixed = quant && !p->uniform_bits;
  const uint32_t uniform = mixed ? 0u : quant ? (uint32_t)p->uniform_bits : 8u;
  const uint8_t* bits = mixed ? p->d_bits : nullptr;
  const uint32_t* off = mixed ? p->d_off : nullptr;
  const LinearTiling tiling = linear_tiling(M, N, K);
  const int64_t tiles = (int64_t)(M / kBM) * (N / kBN);
  if (tiling.whole > 0) {
    auto kernel = !quant  ? k_linear_quantize_pack<DT, GS_LOG2, false, false>
                  : mixed ? k_linear_quantize_pack<DT, GS_LOG2, true, true>
                          : k_linear_quantize_pack<DT, GS_LOG2, false, true>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiling.whole), dim3(kLinThreads), 0, stream, (const char*)x, (const char*)w, M,
                       N, K, lo, hi, uniform, bits, off, (char*)y, words, mn, sc);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || tiling.whole == tiles) return e;
  }
  auto few = [&](auto shape) {
    using S = decltype(shape);
    auto kernel = !quant  ? k_linear_few_tiles<DT, GS_LOG2, false, false, S>
                  : mixed ? k_linear_few_tiles<DT, GS_LOG2, true, true, S>
                          : k_linear_few_tiles<DT, GS_LOG2, false, true, S>;
    const unsigned blocks = (unsigned)((tiles - tiling.whole) * (256 / S::kBM) * (256 / S::kBN));
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(S::kThreads), 0, stream, (const char*)x, (const char*)w, M, N, K, lo, hi,
                       uniform, bits, off, (char*)y, words, mn, sc, (int)tiling.whole);
    return hipGetLastError();
  };
  switch (tiling.cut) {
    case 2: return few(FewBy2{});
    case 4: return few(FewBy4{});
    case 8: return few(FewBy8{});
    case 16: return few(FewBy16<GS_LOG2>{});
    default: return hipErrorInvalidValue;
  }
}

template <int DT>
hipError_t launch_dt(const daf_plan_t* p, const void* x, const void* w, int M, int N, int K, uint64_t seed, void* y,
                     uint32_t* words, float* mn, float* sc, hipStream_t stream) {
  switch (p->group_size) {
    case 32: return launch_gs<DT, 5>(p, x, w, M, N, K, seed, y, words, mn, sc, stream);
    case 64: return launch_gs<DT, 6>(p, x, w, M, N, K, seed, y, words, mn, sc, stream);
    default: return launch_gs<DT, 7>(p, x, w, M, N, K, seed, y, words, mn, sc, stream);
  }
}

}  // namespace

int daf_linear_cut_of(int64_t M, int64_t N, int64_t K, int64_t* whole) {
  const LinearTiling t = linear_tiling(M, N, K);
  *whole = t.whole;
  return t.cut;
}

void daf_linear_few_tile_map(int id, int tiles_m, int tiles_n, int first, int sub_m, int sub_n, int* tm, int* tn) {
  const TileIndex t = few_tile_of_workgroup(id, tiles_m, tiles_n, first, sub_m, sub_n);
  *tm = t.m;
  *tn = t.n;
}

void daf_linear_tile_map(int id, int tiles_m, int tiles_n, int* tm, int* tn) {
  const TileIndex t = tile_of_workgroup(id, tiles_m, tiles_n);
  *tm = t.m;
  *tn = t.n;
}

bool daf_linear_quantize_supported(const daf_plan_t* p, int64_t N, int64_t K, int dtype) {
  if (dtype != DAF_F16 && dtype != DAF_BF16) return false;
  if (p->group_size != 32 && p->group_size != 64 && p->group_size != 128) return false;
  if (N < kBN || N % kBN != 0 || K < kBK || K % kBK != 0 || p->n % N != 0) return false;
  const int64_t M = p->n / N;
  if (M % kBM != 0) return false;
  return M <= (1 << 24) && N <= (1 << 24) && K <= (1 << 24) && (M / kBM) * (N / kBN) < (int64_t)1 << 31;
}

hipError_t daf_launch_linear_quantize_pack(const daf_plan_t* p, const void* x, const void* w, int64_t N, int64_t K,
                                           int dtype, uint64_t seed, void* y, uint32_t* words, float* mn, float* sc,
                                           hipStream_t stream) {
  const int M = (int)(p->n / N);
  if (dtype == DAF_BF16) return launch_dt<kBF16>(p, x, w, M, (int)N, (int)K, seed, y, words, mn, sc, stream);
  return launch_dt<kF16>(p, x, w, M, (int)N, (int)K, seed, y, words, mn, sc, stream);
}
