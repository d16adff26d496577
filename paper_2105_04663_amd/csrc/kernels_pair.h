// bf16 MFMA contraction in 256 x 128 tiles, two workgroups per compute unit: for launches of many tiles with short K, where what a
// workgroup does beside its K loop (finding its problem, first loads, epilogue, drain, the next one's start: 7 to 9 us) is as long as the
// loop.  One workgroup per compute unit (dot_mfma_kernel) leaves the matrix cores idle meanwhile; of two, one multiplies while the other
// loads or stores.
//
// Four waves of 128 x 64 (128 accumulators per lane): a workgroup has 256 registers per lane and 80 KiB of LDS, so 256 x 128 is the largest tile of
// which two fit; in 128 x 128 tiles (dot_mid_kernel) there are twice as many starts and ends.  K in 32-wide tiles through three LDS stages
// of 24 KiB, one barrier per tile: while tile t is multiplied, its neighbour's fragments are read (each lhs fragment into the registers of the
// one just used) and tile t + 3 is loaded into the stage whose fragments were read a tile ago.  Reads and loads are issued one at a time between
// the MFMAs; stages are constants of the code, the last tiles' too, since address arithmetic between MFMAs costs more than the reads themselves.
// What is left of K is one more tile: loads held to the valid K, and each wave clears what lies beyond in the chunks that it loaded, in both
// operands, before the barrier that publishes them.  K tiles in the order and with the instruction of dot_mfma_kernel: results are bit-identical.
//
// Measured (us, dot_mfma_kernel / now): four experts' weight gradients of 256 to 512 x 4096 x 8192 129 / 111; eight of 64 to 128 x 4096 x 4096 82 / 63; eight of
// 150 to 300 x 2048 x 5000 99 / 77; one product of 2048 x 1024 x 4096, both operands K-major, 21.2 / 18.1.  A workgroup of the first takes 12.1 us, two of them on a
// compute unit: 0.6 to find its problem, 1.6 until the first tile is there, 7.6 in the loop (12 tiles; 2.6 of matrix cores), 2.3 for epilogue and
// drain, and 0.4 until the next one.  What bounds it: the latency of loads, of which two tiles are on their way, beside 2.4 TB/s of output
// (matrix cores busy for 46 % of a compute unit's cycles, LDS 14, two fifths of its accesses' cycles bank conflicts; L1 stalled on 47 lines in flight for 38 %).  Six stages
// and one workgroup on a compute unit: 2 to 19 % slower for launches of up to 256 tiles too; plain instead of non-temporal bf16 stores 28 %.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "kernels_basic.h"
#include "kernels_lines.h"
#include "launch.h"
#include "mfma_common.h"
#include "plan.h"
#include "tile_index.h"

namespace gspmd {

constexpr int kPairThreads = 256, kPairStages = 3;
constexpr int kPairPartA = kPairRows * kMfmaBK * 2, kPairPartB = kPairCols * kMfmaBK * 2, kPairStage = kPairPartA + kPairPartB;
constexpr int kPairLds = kPairStages * kPairStage;

template <typename TOut, int LAYOUT>
__global__ __launch_bounds__(kPairThreads, 2) void dot_pair_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
  constexpr int R = kPairStages, kLoads = 6;     // a wave's load instructions of a tile: four of the lhs's part, two of the rhs's
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (wave >> 1) * 128, wn = (wave & 1) * 64;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const int tile = logical_tile(blockIdx.x, gridDim.x);
  const Problem P = lookup_problem(tab, n_prob, tile);
  const int local = tile - P.tile_begin;
  // bands of 1024 rows, the row index running fastest: tiles in flight together share operand panels in L2
  constexpr int kBand = kBandRows / 2;
  const int tiles_m = (P.Mv + kPairRows - 1) / kPairRows;
  const int band = local / (kBand * P.tiles_n), in_band = local - band * kBand * P.tiles_n;
  const int rows_in_band = min(kBand, tiles_m - band * kBand);
  const int m0 = (band * kBand + in_band % rows_in_band) * kPairRows, n_nom = (in_band / rows_in_band) * kPairCols;
  const int n0 = BKC ? n_nom : tile_first_column(n_nom, P.Nv, kPairCols, (P.flags & kProblemMovesBack) != 0);
  const int n_load_end = tile_load_end(n0, n_nom, P.Nv, kPairCols);

  const bf16_bits* a_next = static_cast<const bf16_bits*>(P.A) + (AKM ? static_cast<int64_t>(m0) : static_cast<int64_t>(m0) * P.lda);
  const bf16_bits* b_next = static_cast<const bf16_bits*>(P.B) + (BKC ? static_cast<int64_t>(n0) * P.ldb : static_cast<int64_t>(n0));
  const int64_t a_tile = AKM ? static_cast<int64_t>(kMfmaBK) * P.lda : kMfmaBK, b_tile = BKC ? kMfmaBK : static_cast<int64_t>(kMfmaBK) * P.ldb;
  const int tiles = (P.Kv + kMfmaBK - 1) / kMfmaBK, left = P.Kv % kMfmaBK;

  int a_off[4], b_off[2];
  auto place_loads = [&](int k_valid) {         // in a tile of which `k_valid` k exist
    const int lane = lane_now();                // (as below: nothing that only the last tile needs is kept in registers through the loop)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      a_off[j] = AKM ? mid_km_load_offset<kPairRows>(wave * 4 + j, lane, m0, P.Mv, P.lda, k_valid) : kc_load_offset(wave * 4 + j, lane, m0, P.Mv, P.lda, k_valid);
#pragma unroll
    for (int j = 0; j < 2; ++j)
      b_off[j] = BKC ? kc_load_offset(wave * 2 + j, lane, n0, P.Nv, P.ldb, k_valid) : mid_km_load_offset<kPairCols>(wave * 2 + j, lane, n0, n_load_end, P.ldb, k_valid);
  };
  const uint32_t lds_a = lds0 + wave * 4096, lds_b = lds0 + kPairPartA + wave * 2048;
  auto load_one = [&](int i, int stage) {       // the i-th of this wave's loads of the next tile
    if (i < 4) global_to_lds16(a_next, a_off[i & 3], lds_a + stage * kPairStage + i * 1024);
    else global_to_lds16(b_next, b_off[i & 1], lds_b + stage * kPairStage + (i & 1) * 1024);
    if (i == 3) a_next += a_tile;
    if (i == 5) b_next += b_tile;
  };

  float4_t acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  uint32_t a_from[AKM ? 8 : 1], b_from[BKC ? 1 : 4];            // fragments in stage 0
#pragma unroll
  for (int i = 0; i < (AKM ? 8 : 1); ++i) {
    a_from[i] = lds0 + (AKM ? mid_km_frag_offset<kPairRows>(wm, lane) ^ (i << 5) : kc_frag_offset(wm, lane));
    asm volatile("" : "+v"(a_from[i]));
  }
#pragma unroll
  for (int j = 0; j < (BKC ? 1 : 4); ++j) {
    b_from[j] = lds0 + kPairPartA + (BKC ? kc_frag_offset(wn, lane) : mid_km_frag_offset<kPairCols>(wn, lane) ^ (j << 5));
    asm volatile("" : "+v"(b_from[j]));
  }
  typedef __attribute__((address_space(3))) const u32x4_t lds_u32x4_t;
  auto read_kc = [&](uint32_t at) { return __builtin_bit_cast(bf16x8_t, *(lds_u32x4_t*)(uintptr_t)at); };
  auto read_km = [&](uint32_t at, int row_bytes) {
    short8_t both;
    both.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)at);
    both.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)(at + 4 * row_bytes));
    return __builtin_bit_cast(bf16x8_t, both);
  };
  bf16x8_t fa[8], fb[2][4];                     // of the tile that is multiplied (and the rhs's of the next one)
  auto read_a = [&](int i, int stage) { fa[i] = AKM ? read_km(a_from[AKM ? i : 0] + stage * kPairStage, 2 * kPairRows) : read_kc(a_from[0] + stage * kPairStage + i * 1024); };
  auto read_b = [&](int set, int j, int stage) {
    fb[set][j] = BKC ? read_kc(b_from[0] + stage * kPairStage + j * 1024) : read_km(b_from[BKC ? 0 : j] + stage * kPairStage, 2 * kPairCols);
  };
  auto barrier = [&]() {                        // (the compiler moves no LDS access across it)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // beyond the valid K, in the chunks of the last tile that this wave has loaded (into `stage`), both operands: the padding may hold anything
  auto clear_beyond = [&](int stage) {
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    asm volatile("" ::: "memory");
    const int lane = lane_now();
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const bool kmajor = i < 4 ? AKM : !BKC;
      const int q = i < 4 ? wave * 4 + i : wave * 2 + i - 4;
      const int k = kmajor ? (i < 4 ? q * 2 + (lane >> 5) : q * 4 + (lane >> 4)) : ((lane & 3) ^ swz_a(q * 16 + (lane >> 2))) * 8;
      __attribute__((address_space(3))) u32x4_t* at = (__attribute__((address_space(3))) u32x4_t*)(uintptr_t)((i < 4 ? lds_a + i * 1024 : lds_b + (i - 4) * 1024) + stage * kPairStage + lane * 16);
      *at = mask_tail8(*at, kmajor ? (k < left ? 8 : 0) : left - k);
    }
  };
  // Tile `u` (modulo 6) multiplied, between the MFMAs the next one's fragments read (from the stage behind its own) and, if there is one, the tile
  // three further on loaded.  `set` u % 2, stage u % 3.
  auto multiply = [&](auto u_tag, bool loads) {
    constexpr int u = decltype(u_tag)::value, set = u & 1, here = u % R, next = (u + 1) % R;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      const int i = q >> 2, j = i & 1 ? 3 - (q & 3) : q & 3;    // back and forth: every MFMA shares an operand with the one before it
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if ((q & 3) == 3) read_a(i, next);
      if ((q & 3) == 1 && i < 4) read_b(set ^ 1, i, next);
      if (loads && (q & 3) == 2 && i < kLoads) load_one(i, here);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // waits until the tile after this one has landed, `after` younger tiles being on their way, and this wave's fragment reads are over
  auto landed = [&](int after) {
    if (after >= 2) __builtin_amdgcn_s_waitcnt(waitcnt_imm(2 * kLoads, 0));
    else if (after == 1) __builtin_amdgcn_s_waitcnt(waitcnt_imm(kLoads, 0));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    barrier();
  };

  if (tiles > 0) {
    place_loads(tiles == 1 && left ? left : kMfmaBK);
    for (int s = 0; s < min(tiles, R); ++s) {
      if (left && s > 0 && s == tiles - 1) place_loads(left);
#pragma unroll
      for (int i = 0; i < kLoads; ++i) load_one(i, s);
    }
    if (left && tiles == 1) clear_beyond(0);
    landed(min(tiles, R) - 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) read_b(0, j, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) read_a(i, 0);
    int k = 0;                                  // tile being multiplied
    auto whole = [&](auto u_tag) {              // whose successors are whole and there
      landed(R - 2);
      multiply(u_tag, true);
    };
    for (; k + 6 + R < tiles; k += 6) {
      whole(std::integral_constant<int, 0>{});
      whole(std::integral_constant<int, 1>{});
      whole(std::integral_constant<int, 2>{});
      whole(std::integral_constant<int, 3>{});
      whole(std::integral_constant<int, 4>{});
      whole(std::integral_constant<int, 5>{});
    }
    const int rest = tiles - k;                 // 1 .. 9 tiles, the last of which may be partial
    auto ending = [&](auto u_tag, auto next) {
      constexpr int u = decltype(u_tag)::value;
      if (left && u + 2 == rest) clear_beyond((u + 1) % R);
      if (left && u + R + 1 == rest) place_loads(left);
      landed(min(rest, u + R) - (u + 2));
      multiply(u_tag, u + R < rest);
      if constexpr (u < 8)
        if (u + 1 < rest) next(std::integral_constant<int, u + 1>{}, next);
    };
    ending(std::integral_constant<int, 0>{}, ending);
  }

  // ---- epilogue
  GSPMD_GLOBAL TOut* const C = (GSPMD_GLOBAL TOut*)P.C;
  constexpr int kAtOnce = sizeof(TOut) == 2 ? 8 : 4;
  static_assert(4 * line_slice<TOut>(kAtOnce) <= kPairLds, "");
  __syncthreads();                              // every wave's fragment reads are over
  store_lines<TOut, 8, kAtOnce, sizeof(TOut) == 2 ? kLinesPast : kLinesPlain>(smem + wave * line_slice<TOut>(kAtOnce), C, P, m0 + wm, n0 + wn, m0 + kPairRows <= P.Mv && n0 + kPairCols <= P.Nv, epilogue, lane,
                                [&](int i, int j) { return acc[i][j]; });
  // zeros of the static block below the last row tile, over this tile's columns (what lies further down, and whole tile
  // columns of padding, the fill kernel clears), and right of a tile that was moved back
  const int m_done = min(m0 + kPairRows, P.Mv), moved_end = n0 + kPairCols, col_end = min(n_nom + kPairCols, P.Ns);
  if (n0 < n_nom) zero_block<kPairThreads, TOut>(C, P.ldc, m0, m_done, moved_end, col_end, t);
  if (m_done == P.Mv) {
    zero_block<kPairThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), n0, min(moved_end, P.Ns), t);
    if (n0 < n_nom) zero_block<kPairThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), moved_end, col_end, t);
  }
}

template <int LAYOUT, typename TOut>
inline bool launch_dot_pair_as(const MfmaLaunch& l, hipStream_t stream) {
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::call_once(once[dev], [dev] {
    ok[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&dot_pair_kernel<TOut, LAYOUT>), hipFuncAttributeMaxDynamicSharedMemorySize, kPairLds) == hipSuccess;
  });
  if (!ok[dev]) return false;
  hipLaunchKernelGGL((dot_pair_kernel<TOut, LAYOUT>), dim3(static_cast<unsigned>(l.tiles)), dim3(kPairThreads), kPairLds, stream, *l.inl, l.tab, l.n_prob, l.epilogue);
  return hipGetLastError() == hipSuccess;
}

template <int LAYOUT>
bool launch_dot_pair_layout(const MfmaLaunch& l, int32_t out_dtype, hipStream_t stream) {
  return out_dtype == GSPMD_F32 ? launch_dot_pair_as<LAYOUT, float>(l, stream) : launch_dot_pair_as<LAYOUT, bf16_bits>(l, stream);
}

}  // namespace gspmd
