// The linear layer with a quantizing epilogue, for outputs that are too few tiles of 256 x 256 to occupy the chip.
//
// A tile of 256 x 256 takes one compute unit ~1.17 us per 64 values of k whatever the other 255 do, so a product of
// 512 x 5120 x 1792 (40 tiles) takes as long as one of six times its size.  Here the tiles are 128 x 256, 128 x 128, 64 x 128 or
// 64 x 64 (32 x 128 where a group is 128 elements): 2, 4, 8 or 16 out of one of 256 x 256, on 4 waves and with one wave per SIMD:
//   - what bounds it is the LDS (128 x 128: 64 KB of operand reads and 32 KB of arriving tiles per step, 750 cycles at
//     128 bytes per cycle beside 512 cycles of matrix instructions; the others have more reads for each of
//     those, 128 x 256 fewer) and, the smaller the product, the way of the operands
//     from memory.  So STAGES steps of operands are on their way or waiting in LDS (loads straight into LDS,
//     whole cache lines, counted waits), and a step's operands are read into registers one step ahead, which frees
//     a stage as soon as it has been read and leaves the matrix instructions nothing to wait for;
//   - the workgroups of a die get consecutive tiles of panels of four tile rows, so that they share operand rows in its cache.
// Large products take these tiles for what whole rounds of 256 workgroups leave over.
#pragma once
#include "linear_common.h"

namespace {

template <int BM, int BN, int WAVES_M, int WAVES_N, int STAGES>
struct FewTiles {
  static constexpr int kBM = BM, kBN = BN, kWavesM = WAVES_M, kWavesN = WAVES_N, kStages = STAGES;
  static constexpr int kWaves = WAVES_M * WAVES_N, kThreads = kWaves * kWave;
  static constexpr int kMB = BM / WAVES_M / 32, kNB = BN / WAVES_N / 32;       // blocks of 32 x 32 of a wave
  static constexpr int kRowBytes = 128;                                        // 64 values of k: one cache line
  static constexpr int kStageBytes = (BM + BN) * kRowBytes;                    // W's rows, then x's
  static constexpr int kLoads = (BM + BN) / 8 / kWaves;                        // of 8 rows, per wave and step
  static_assert(kMB * WAVES_M * 32 == BM && kNB * WAVES_N * 32 == BN && kLoads * kWaves * 8 == BM + BN, "tile shape");
  static_assert(kWaves % 2 == 0 && BN % 8 == 0, "a wave's rows keep their place modulo 16");
  static_assert(STAGES >= 3 && (STAGES - 1) * kLoads <= 63 && STAGES * kStageBytes <= 160 * 1024, "stages");
};
// By the number of 256 x 256 tiles they cut one into.
using FewBy2 = FewTiles<128, 256, 2, 2, 3>;
using FewBy4 = FewTiles<128, 128, 2, 2, 4>;
using FewBy8 = FewTiles<64, 128, 2, 2, 6>;
template <int GS_LOG2>
using FewBy16 = typename std::conditional<GS_LOG2 == 7, FewTiles<32, 128, 1, 4, 6>, FewTiles<64, 64, 2, 2, 8>>::type;

// blockIdx -> tile.  The 256 x 256 tiles from position `first` of the sequence (tile_of_position) to its end, each cut
// into sub_m x sub_n; every die (blockIdx mod 8) takes a run of consecutive ones.  Visits every tile once.
__host__ __device__ inline TileIndex few_tile_of_workgroup(int id, int tiles_m, int tiles_n, int first, int sub_m, int sub_n) {
  constexpr int kDies = 8, kPanel = 4;
  const int subs = sub_m * sub_n, total = (tiles_m * tiles_n - first) * subs, each = total / kDies, more = total % kDies;
  const int die = id % kDies;
  const int pos = die * each + (die < more ? die : more) + id / kDies;
  const int sub = pos % subs;
  TileIndex t = tile_of_position(first + pos / subs, tiles_m, tiles_n, kPanel);
  t.m = t.m * sub_m + sub % sub_m;
  t.n = t.n * sub_n + sub / sub_m;
  return t;
}

template <int N>
__device__ __forceinline__ void wait_loads_and_reads() {               // all but N loads into LDS, all LDS reads
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

template <int DT, int GS_LOG2, bool MIXED, bool QUANT, class S>
__global__ __launch_bounds__(S::kThreads, 1) void k_linear_few_tiles(
    const char* __restrict__ x, const char* __restrict__ w, int M, int N, int K, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t uniform_b, const uint8_t* __restrict__ bits, const uint32_t* __restrict__ off, char* __restrict__ y,
    uint32_t* __restrict__ words, float* __restrict__ out_min, float* __restrict__ out_scale, int first) {
  constexpr int kMB = S::kMB, kNB = S::kNB, kStages = S::kStages;
  __shared__ __align__(1024) char lds[kStages * S::kStageBytes];
  const int t = threadIdx.x, lane = t & (kWave - 1);
  const int uw = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = uw % S::kWavesM, wn = uw / S::kWavesM;
  const int li = lane & 31, lg = lane >> 5;

  const TileIndex ti = few_tile_of_workgroup((int)blockIdx.x, M / 256, N / 256, first, 256 / S::kBM, 256 / S::kBN);
  const int64_t m0 = (int64_t)ti.m * S::kBM, n0 = (int64_t)ti.n * S::kBN;
  const int steps = K / 64;
  const int64_t row_bytes = (int64_t)K * 2;

  // Load i of a wave: 8 rows of W (first kBN rows of a stage) or of x.  Row r's 16-byte piece p goes to place
  // p ^ (r / 2 mod 8): no bank conflicts when 32 consecutive rows are read.
  const uint32_t piece = (uint32_t)((lane & 7) ^ ((lane >> 4) | ((uw & 1) << 2)));
  const uint32_t l_off = (uint32_t)(lane >> 3) * (uint32_t)row_bytes + (piece << 4);
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds);
  const char* src[S::kLoads];
#pragma unroll
  for (int i = 0; i < S::kLoads; ++i) {
    const int row = (i * S::kWaves + uw) * 8;
    src[i] = uniform_pointer(row < S::kBN ? w + (n0 + row) * row_bytes : x + (m0 + row - S::kBN) * row_bytes);
  }
  // Load i of step `s` into stage `st`.  Past the end the last step again (never used): the counts stay the same.
  auto fetch = [&](int i, int s, int st) {
    load_to_lds(lds0 + (uint32_t)(st * S::kStageBytes + (i * S::kWaves + uw) * 1024), l_off, src[i]);
    src[i] += s + 1 < steps ? S::kRowBytes : 0;
  };

  const char *pa[4], *pb[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int col = ((2 * ks + lg) ^ ((li >> 1) & 7)) << 4;
    pa[ks] = lds + (wn * kNB * 32 + li) * S::kRowBytes + col;
    pb[ks] = lds + (S::kBN + wm * kMB * 32 + li) * S::kRowBytes + col;
  }
  f32x16 acc[kMB][kNB];
#pragma unroll
  for (int i = 0; i < kMB; ++i)
#pragma unroll
    for (int j = 0; j < kNB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  u32x4 a[2][kNB][4], b[2][kMB][4];                       // operands of even and odd steps
  constexpr int kReads = 4 * (kNB + kMB), kMfma = 4 * kNB * kMB;
  auto read = [&](int q, int parity, int st) {            // read q of a step: by k, W's blocks and then x's
    const int ks = q / (kNB + kMB), j = q % (kNB + kMB);
    const int at = st * S::kStageBytes;
    if (j < kNB) a[parity][j][ks] = *reinterpret_cast<const u32x4*>(pa[ks] + at + j * 32 * S::kRowBytes);
    else b[parity][j - kNB][ks] = *reinterpret_cast<const u32x4*>(pb[ks] + at + (j - kNB) * 32 * S::kRowBytes);
  };

  constexpr int kGs = 1 << GS_LOG2, kWaveN = kNB * 32;
  constexpr int kShare = kGs > kWaveN ? kGs / kWaveN : 1;               // waves (along n) that share a group
  constexpr int kGroups = kGs > kWaveN ? 1 : kWaveN / kGs, kBlocksPerGroup = kNB / kGroups;
  const int64_t m_lane = m0 + wm * kMB * 32 + li, n_lane = n0 + wn * kWaveN + lg * 16;
  // The lane's groups' widths and offsets first, one load each for those of a row: behind the stores of y a wait for them would be one
  // for those too.  (Groups of 32, bfloat16, one load a group / a row: 2048 x 1024 x 4096 27.9 / 26.1 us, 1792 x 4096 x 1344 31.0 / 29.9; group by
  // group where they are used 26.7 and 31.0.)
  [[maybe_unused]] RowGroups<kGroups> row[kMB];
  if constexpr (QUANT && MIXED) {
#pragma unroll
    for (int i = 0; i < kMB; ++i) row[i] = row_groups<kGroups>(bits, off, ((m_lane + i * 32) * N + n0 + wn * kWaveN) >> GS_LOG2);
  }

#pragma unroll
  for (int st = 0; st < kStages; ++st)
#pragma unroll
    for (int i = 0; i < S::kLoads; ++i) fetch(i, st, st);
  wait_loads_and_reads<(kStages - 1) * S::kLoads>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int q = 0; q < kReads; ++q) read(q, 0, 0);

  int st = 0;                                             // stage of step s
  auto step = [&](auto parity, int s) {
    constexpr int P = decltype(parity)::value;
    // Every wave has read step s out of its stage, and step s + 1 has arrived for all: kStages - 2 steps stay on their way.
    wait_loads_and_reads<(kStages - 2) * S::kLoads>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    const int next = st + 1 < kStages ? st + 1 : 0;
#pragma unroll
    for (int q = 0; q < kMfma; ++q) {
      const int ks = q / (kNB * kMB), j = q % (kNB * kMB);
      acc[j / kNB][j % kNB] = mfma16<DT>(a[P][j % kNB][ks], b[P][j / kNB][ks], acc[j / kNB][j % kNB]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = q * S::kLoads / kMfma; i < (q + 1) * S::kLoads / kMfma; ++i) fetch(i, s + kStages, st);
#pragma unroll
      for (int r = q * kReads / kMfma; r < (q + 1) * kReads / kMfma; ++r) read(r, P ^ 1, next);
      __builtin_amdgcn_sched_barrier(0);
    }
    st = next;
  };
  int s = 0;
  for (; s + 1 < steps; s += 2) {
    step(std::integral_constant<int, 0>{}, s);
    step(std::integral_constant<int, 1>{}, s + 1);
  }
  if (s < steps) step(std::integral_constant<int, 0>{}, s);
  wait_loads_and_reads<0>();

  // ---- epilogue ----
  float xf[kMB][kNB][16], gmn[kMB][kGroups], gmx[kMB][kGroups];
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb) {
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      uint32_t yv[8];
      block_row<DT>(acc[mb][nb], yv);
      char* dst = y + ((m_lane + mb * 32) * N + n_lane + nb * 32) * 2;
      *reinterpret_cast<u32x4*>(dst) = u32x4{yv[0], yv[1], yv[2], yv[3]};
      *reinterpret_cast<u32x4*>(dst + 16) = u32x4{yv[4], yv[5], yv[6], yv[7]};
      if (!QUANT) continue;                                            // the product alone
      float mn, mx;
      widen_row<DT>(yv, xf[mb][nb], mn, mx);
      const int gi = nb / kBlocksPerGroup;
      gmn[mb][gi] = nb % kBlocksPerGroup ? vmin(gmn[mb][gi], mn) : mn;
      gmx[mb][gi] = nb % kBlocksPerGroup ? vmax(gmx[mb][gi], mx) : mx;
    }
  }
  if (!QUANT) return;
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      gmn[mb][gi] = both_halves_min(gmn[mb][gi]);
      gmx[mb][gi] = both_halves_max(gmx[mb][gi]);
    }
  if constexpr (kShare > 1) {
    float2(*stat)[S::kBM] = reinterpret_cast<float2(*)[S::kBM]>(lds);    // [wave along n][row]
    __syncthreads();                                                     // every wave's loads have landed, its reads are done
    if (lg == 0) {
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) stat[wn][(wm * kMB + mb) * 32 + li] = make_float2(gmn[mb][0], gmx[mb][0]);
    }
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
      for (int q = 0; q < kShare; ++q) {
        const float2 o = stat[wn / kShare * kShare + q][(wm * kMB + mb) * 32 + li];
        gmn[mb][0] = vmin(gmn[mb][0], o.x);
        gmx[mb][0] = vmax(gmx[mb][0], o.y);
      }
  }
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb) {
    const int64_t m = m_lane + mb * 32;
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
      const int64_t g = (m * N + n0 + wn * kWaveN + gi * kGs) >> GS_LOG2;
      const uint32_t gb = MIXED ? (uint32_t)row[mb].b.of[gi] : uniform_b;
      const uint32_t woff = MIXED ? row[mb].off.of[gi] : (uint32_t)(g * (int64_t)((kGs * uniform_b) >> 5));
      const GroupScale gs = group_scale(gmn[mb][gi], gmx[mb][gi], gb);
      if (lg == 0 && wn % kShare == 0) {
        out_min[g] = gs.mn;
        out_scale[g] = gs.scale;
      }
      const LinearGroup group = linear_group(gs, gb, words + woff);
#pragma unroll
      for (int q = 0; q < kBlocksPerGroup; ++q) {
        const int nb = gi * kBlocksPerGroup + q;
        quantize_row(xf[mb][nb], group, (uint32_t)(wn % kShare * kWaveN + q * 32 + lg * 16), m * N + n_lane + nb * 32,
                     seed_lo, seed_hi, lg);
      }
    }
  }
}

}  // namespace
