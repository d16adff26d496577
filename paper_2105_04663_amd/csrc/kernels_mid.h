// bf16 MFMA contraction in 128 x 128 tiles, one or two workgroups per compute unit: for launches that 256 x 256 tiles (one
// workgroup per compute unit, 9 us beside its K loop) leave waiting or idle -- few output tiles, short K -- and for sums over
// a contracting mesh dimension, which it forms without a workspace: a workgroup takes the members' K ranges one after
// the other (without a break where they are alike: 2048 x 8192 x 2048 over 4 members 66.8 -> 62.9 us) and adds each member's finished product to a second set of accumulators, so the sum is ((p0 + p1) + p2) + ..
// in fp32 as everywhere else.  Products take their 32-wide K tiles in the order and with the instruction of
// dot_mfma_kernel: results are bit-identical to it.  Operands at multiples of 4 bytes (see there).
//
// What bounds it: what a compute unit draws from L2 and beyond, 16 KiB per 32-wide K tile for 256 cycles of the matrix cores: the loads
// alone take 190 ns per tile on a full chip, 135 on few compute units, a tile with everything 205 (400 for two workgroups).  So:
// a K step is 64 wide, two tiles.  Of a K-contiguous operand each tile holds half of the 128 rows, 64 k of each, whole lines of
// 128 bytes (in [128][32 k] tiles every line comes twice: the loads alone 236 ns); of a K-major operand 32 k rows, [32 k][128], read
// with the transpose read.  A wave issues one fragment read or load after each MFMA (all of a tile's ahead of its MFMAs: 240 ns), and
// the stages come round every five steps, so that their places are constants of the code.  One barrier per step.  With one workgroup
// on a compute unit ten stages (160 KiB), loads six tiles ahead; with two five stages each, four ahead.
// Measured (us, with 32-wide steps / now): 2048 x 8192 x 2048 73.5 / 62, 512 x 8192 x 512 67.7 / 45, 2048 x 4096 x 4096 73 / 60, 2112 x 8000 x
// 2112 118 / 90, both K-contiguous 127 / 92.  2048 x 8192 x 2048 over 4 members: 64 with operands in the memory-side cache, 82 from HBM.
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

constexpr int kMidPart = kMidTile * kMfmaBK * 2;      // 8 KiB: one operand's 32-wide K tile
constexpr int kMidStage = 2 * kMidPart;
// LDS stages with one and with two workgroups on a compute unit, and how many tiles ahead of the multiplication loads are issued
template <int PER_CU> constexpr int mid_stages() { return PER_CU == 1 ? 10 : 5; }
template <int PER_CU> constexpr int mid_ahead() { return PER_CU == 1 ? 6 : 4; }
constexpr int kStorePast = 256;                       // beside the epilogue in a launch's arguments: bf16 outputs past all caches
constexpr int kMidUnroll = 5;                         // K steps after which the stages come round: their places are then constants of the code

// STAGED: the variant for operands at odd element addresses, which direct loads do not take: a tile's chunks are loaded into registers two
// half steps before they are put where the direct load would have put them, and K-major operands' last tiles are moved back so that
// every chunk is whole.  Bound by the address unit, 64 cycles for a KiB at an odd address (both operands: 430 ns per 32-wide
// tile, one 270).  Measured (us, before in 256 x 256 staged tiles or dot_split_kernel / now): 601 x 1203 x 697, six of them 49.5 / 17.5,
// 4999 x 576 x 1193 28.1 / 15.2, 152 x 209 x 1094, 32 of them 23.7 / 16.6.
template <typename TOut, int LAYOUT, bool CHAIN, int PER_CU, bool STAGED>
__global__ __launch_bounds__(kMidThreads, CHAIN && PER_CU == 1 ? 1 : 2)   // (one: the sums' accumulators take the other half of the registers)
 void dot_mid_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
  static_assert(!(STAGED && CHAIN) && (!STAGED || PER_CU == 2), "");
  constexpr int R = mid_stages<PER_CU>(), L = mid_ahead<PER_CU>();
  static_assert(2 * kMidUnroll % R == 0, "the loop's stages come round");
  // A tile's load is issued in the half step L tiles before it is multiplied, into a stage whose last reads every wave has behind it: the
  // reads of the K step before the current one (those of the step itself too, where the barrier waits for them).
  constexpr bool kReadsDone = L > R - 3;
  static_assert(L % 2 == 0 && L >= 4 && L < R, "loads run ahead by whole K steps, and a stage is free before it is filled");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const int tile = logical_tile(blockIdx.x, gridDim.x);
  const int which = lookup_problem_index(tab, n_prob, tile);
  Problem P = problem_at(tab, which);
  const int local = tile - P.tile_begin;
  // bands of kBandRows tile rows, the row index running fastest: tiles in flight together share operand panels in L2
  const int tiles_m = (P.Mv + kMidTile - 1) / kMidTile;
  const int band = local / (kBandRows * P.tiles_n), in_band = local - band * kBandRows * P.tiles_n;
  const int rows_in_band = min(kBandRows, tiles_m - band * kBandRows);
  const int m_nom = (band * kBandRows + in_band % rows_in_band) * kMidTile, n_nom = (in_band / rows_in_band) * kMidTile;
  const int n0 = BKC ? n_nom : STAGED ? min(n_nom, P.Nv - kMidTile) : tile_first_column(n_nom, P.Nv, kMidTile, (P.flags & kProblemMovesBack) != 0);
  const int n_load_end = tile_load_end(n0, n_nom, P.Nv, kMidTile);
  const int m0 = STAGED && AKM ? min(m_nom, P.Mv - kMidTile) : m_nom;
  const int members = CHAIN ? max(P.join_count, 1) : 1;
  // Members that are alike follow each other without a break: the loads of the next one are under way while this one's last steps are
  // multiplied (those with something left of K in the loop that is not unrolled, so only short ones).  Others are taken one by one.
  const bool run_on = CHAIN && (P.flags & kProblemRunsOn) != 0;
  // A sum's kernel with two workgroups on a compute unit has 256 registers, and its loop takes them all: what only a member's start, its rest of K and the
  // epilogue need is worked out there.  Kept from the start, 7 to 17 registers were spilled and reloaded for every member (us, spilled / now: 2048 x 2048 x 8192 over
  // 2 members, two groups 64.0 / 61.1, 2048 x 8192 x 4096 over 4 128.0 / 123.4, float32 results of 3072 x 2000 x 3072 over 2 59.7 / 55.8; 31 sums of all layouts 1.00 to 1.07 times as fast).
  constexpr bool kFewRegisters = CHAIN && PER_CU == 2;
  auto lane_here = [&]() { return kFewRegisters ? lane_now() : lane; };

  float4_t acc[4][4], sum[CHAIN ? 4 : 1][CHAIN ? 4 : 1];
  // Fragment addresses.  LDS offsets in instructions have 16 bits: stages are addressed from a register per four of them (with five
  // stages: one for the first four, one for the last).  A K-contiguous operand's register says which half of the rows this wave reads, and
  // with five stages the second one stands for a step whose second tile is in stage 0 again.
  constexpr int kGroups = R == 10 ? 3 : 2;
  const int a_half = wm >> 6, b_half = wn >> 6;
  uint32_t a_reg[kGroups][AKM ? 4 : 2], b_reg[kGroups][BKC ? 2 : 4];
  auto half_at = [&](int g, int half) { return R == 5 && g == 1 ? (half ? 0 : 4) : g * 4 + half; };
#pragma unroll
  for (int g = 0; g < (kFewRegisters ? 1 : kGroups); ++g) {
#pragma unroll
    for (int i = 0; i < (AKM ? 4 : 2); ++i) {
      a_reg[g][i] = lds0 + (AKM ? (mid_km_frag_offset(wm, lane) ^ (i << 5)) + g * 4 * kMidStage : (kc_half_frag_offset(0, lane) ^ (i * 64)) + half_at(g, a_half) * kMidStage);
      asm volatile("" : "+v"(a_reg[g][i]));
    }
#pragma unroll
    for (int i = 0; i < (BKC ? 2 : 4); ++i) {
      b_reg[g][i] = lds0 + kMidPart + (BKC ? (kc_half_frag_offset(0, lane) ^ (i * 64)) + half_at(g, b_half) * kMidStage : (mid_km_frag_offset(wn, lane) ^ (i << 5)) + g * 4 * kMidStage);
      asm volatile("" : "+v"(b_reg[g][i]));
    }
  }
  // where registers are few the second group's are worked out for every member
  auto place_groups = [&]() {
    if constexpr (kFewRegisters) {
      auto from = [&](uint32_t first, bool kmajor, int half) {
        uint32_t at;
        asm volatile("v_add_u32_e32 %0, %1, %2" : "=v"(at) : "s"(kmajor ? 4 * kMidStage : (half_at(1, half) - half_at(0, half)) * kMidStage), "v"(first));
        return at;
      };
#pragma unroll
      for (int i = 0; i < (AKM ? 4 : 2); ++i) a_reg[1][i] = from(a_reg[0][i], AKM, a_half);
#pragma unroll
      for (int i = 0; i < (BKC ? 2 : 4); ++i) b_reg[1][i] = from(b_reg[0][i], !BKC, b_half);
    }
  };
  typedef __attribute__((address_space(3))) const u32x4_t lds_u32x4_t;
  auto read_kc = [&](uint32_t at) { return __builtin_bit_cast(bf16x8_t, *(lds_u32x4_t*)(uintptr_t)at); };
  auto read_km = [&](uint32_t at) {
    short8_t both;
    both.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)at);
    both.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(uintptr_t)(at + 4 * 256));
    return __builtin_bit_cast(bf16x8_t, both);
  };
  bf16x8_t fa[2][4], fb[2][4];                  // fragments of two 32-wide tiles: one being multiplied, the next being read
  auto multiply = [&](int set) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
  };

  auto add_member = [&](bool first) {
    if constexpr (CHAIN) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[i][j] = first ? acc[i][j] : sum[i][j] + acc[i][j];
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  };

  for (int member = 0; member < (run_on ? 1 : members); ++member) {
    if (CHAIN && member > 0) {
      P = problem_at(tab, which + member);
      __syncthreads();                          // every wave has read the last tile of the member before
    }
    clear();
    place_groups();
    const int64_t a_first = AKM ? static_cast<int64_t>(m0) : static_cast<int64_t>(m0) * P.lda, b_first = BKC ? static_cast<int64_t>(n0) * P.ldb : static_cast<int64_t>(n0);
    const bf16_bits* a_base = static_cast<const bf16_bits*>(P.A) + a_first;
    const bf16_bits* b_base = static_cast<const bf16_bits*>(P.B) + b_first;
    const int64_t a_tile = AKM ? static_cast<int64_t>(kMfmaBK) * P.lda : kMfmaBK, b_tile = BKC ? kMfmaBK : static_cast<int64_t>(kMfmaBK) * P.ldb;
    // of K after the whole 64-wide steps; of members that follow on, the last one may have less K than the others
    const int left = P.Kv % (2 * kMfmaBK), last_k = run_on ? problem_at(tab, which + members - 1).Kv : P.Kv, last_left = last_k % (2 * kMfmaBK);
    // What is left is one more step, its loads held to the valid K and its fragments cleared beyond; only where a chunk of eight k that is
    // partly valid may reach past its row's end, and where registers are short, it is taken after the loop (below): the partial tile through
    // registers, a whole one before it straight to LDS, both on their way together.  (One after the other through registers, with two workgroups on a
    // compute unit: 1500 x 3000 x 4096 over 8 members 71.1 us, now 67.4; 2000 x 1500 x 3000 over 4 41.2, 38.2.)
    const bool masked = !STAGED && !(CHAIN && PER_CU == 2) && (left | last_left) > 0 && ((left | last_left) % 8 == 0 || ((AKM || !loose_rows(P.A, P.lda)) && (!BKC || !loose_rows(P.B, P.ldb))));
    const int own = (P.Kv / (2 * kMfmaBK) + (masked && left > 0 ? 1 : 0)) * 2;       // a member's tiles
    const int last_own = (last_k / (2 * kMfmaBK) + (masked && last_left > 0 ? 1 : 0)) * 2;
    const int tiles = run_on ? own * (members - 1) + last_own : own;
    int a_off[2][2], b_off[2][2];               // this wave's two load instructions of each operand's part, in even and odd tiles
    auto place_loads = [&](int k_valid) {       // in a step of which `k_valid` k exist
      const int lane = lane_here();
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int q = wave * 2 + j, here = h == 0 || k_valid <= kMfmaBK ? min(k_valid, kMfmaBK) : k_valid - kMfmaBK;
          a_off[h][j] = AKM ? mid_km_load_offset(q, lane, m0, P.Mv, P.lda, here) : mid_kc_load_offset(q, lane, h, m0, P.Mv, P.lda, k_valid);
          b_off[h][j] = BKC ? mid_kc_load_offset(q, lane, h, n0, P.Nv, P.ldb, k_valid) : mid_km_load_offset(q, lane, n0, n_load_end, P.ldb, here);
        }
    };
    int64_t a_go, b_go;                         // how far a K-major operand's next tile is
    auto place_whole = [&]() {
      place_loads(2 * kMfmaBK);
      a_go = a_tile;
      b_go = b_tile;
    };
    place_whole();
    // the last step's: of a K-major operand with nothing left in the step's second half, the first half's rows once more
    int left_loading = left, left_adding = left;          // of the members being loaded and multiplied
    auto place_last = [&]() {
      if (left_loading == 0) return;
      place_loads(left_loading);
      if (left_loading <= kMfmaBK) a_go = b_go = 0;
    };
    const bf16_bits *a_next = a_base, *b_next = b_base;
    const uint32_t lds_wave = lds0 + wave * 2048;
    int to_load = own / 2, loading = 0, adding = 0, to_add = own / 2;                     // K steps of the members being loaded and multiplied that are to come
    bool to_add_first = true;
    u32x4_t held[STAGED ? 2 : 1][STAGED ? 4 : 1];                            // STAGED: this wave's chunks of an even and an odd tile on their way
    // the i-th of this wave's four load instructions of an even (h 0) or odd tile, into stage `at` (STAGED: into registers)
    auto issue_one = [&](int h, int i, int at) {
      if constexpr (STAGED) {
        typedef uint32_t any_t __attribute__((ext_vector_type(4), aligned(2)));
        typedef GSPMD_GLOBAL const unsigned char* gbytes;
        held[h][i] = i < 2 ? *(GSPMD_GLOBAL const any_t*)((gbytes)a_next + static_cast<uint32_t>(a_off[h][i & 1])) : *(GSPMD_GLOBAL const any_t*)((gbytes)b_next + static_cast<uint32_t>(b_off[h][i & 1]));
      } else if (i < 2) {
        global_to_lds16(a_next, a_off[h][i & 1], lds_wave + at * kMidStage + (i & 1) * 1024);
      } else {
        global_to_lds16(b_next, b_off[h][i & 1], lds_wave + at * kMidStage + kMidPart + (i & 1) * 1024);
      }
      if (i == 3) {
        if (AKM) a_next += a_go;
        else if (h == 1) a_next += 2 * kMfmaBK;
        if (!BKC) b_next += b_go;
        else if (h == 1) b_next += 2 * kMfmaBK;
        if (h == 1) --to_load;
        if (CHAIN && h == 1 && run_on && to_load == 0) {                      // on to the next member
          if (masked) place_whole();
          ++loading;
          to_load = (loading == members - 1 ? last_own : own) / 2;
          left_loading = loading == members - 1 ? last_left : left;
          if (loading < members) {
            const Problem Q = problem_at(tab, which + loading);
            a_next = static_cast<const bf16_bits*>(Q.A) + a_first;
            b_next = static_cast<const bf16_bits*>(Q.B) + b_first;
          }
        }
      }
    };
    auto put_one = [&](int h, int i, int at) {  // STAGED: a chunk that has arrived, into stage `at`
      if constexpr (STAGED)
        *(__attribute__((address_space(3))) u32x4_t*)(uintptr_t)(lds_wave + at * kMidStage + (i >> 1) * kMidPart + (i & 1) * 1024 + lane * 16) = held[h][i];
    };
    auto step_done = [&]() {                    // a K step has been multiplied
      --to_add;
      if (CHAIN && run_on && to_add == 0) {
        add_member(to_add_first);
        clear();
        to_add_first = false;
        ++adding;
        to_add = (adding == members - 1 ? last_own : own) / 2;
        left_adding = adding == members - 1 ? last_left : left;
      }
    };
    // Fragment i (rhs 0..3, then lhs 0..3) of half h of a K step whose first tile is in stage s0, into set h.  A K-contiguous operand's
    // rows are all in the tile of their half of the 128 rows, 64 k each; a K-major operand's k rows in the tile of their half of the step.
    // `fixed`: s0 is a constant, and so is what is added to the registers.
    auto read_one = [&](int h, int i, int s0, bool fixed) {
      const int s_km = s0 + h >= R ? s0 + h - R : s0 + h;
      auto place = [&](int s, uint32_t (&first), uint32_t (&of_group)) { return fixed ? of_group + (R == 5 && s == 4 ? 0 : (s & 3) * kMidStage) : first + s * kMidStage; };
      auto km = [&](auto& reg, int x) { return place(s_km, reg[0][x], reg[s_km >> 2][x]); };
      auto kc = [&](auto& reg, int half) {                 // the tile of this wave's half: the step's second one may be in stage 0 again
        if (fixed) return place(s0, reg[0][h], reg[s0 >> 2][h]);
        const int s = s0 + half;
        return reg[0][h] + (s >= R ? s - R - half : s0) * kMidStage;
      };
      if (i < 4) fb[h][i] = BKC ? read_kc(kc(b_reg, b_half) + i * 2048) : read_km(km(b_reg, BKC ? 0 : i));
      else fa[h][i - 4] = AKM ? read_km(km(a_reg, AKM ? i - 4 : 0)) : read_kc(kc(a_reg, a_half) + (i - 4) * 2048);
    };
    // Half a K step: the MFMAs of fragment set `set`, and between them, one at a time, the reads of the next half's fragments (of the
    // step in stage s0) and the loads of the tile L further on (into stage `to`).
    // STAGED: a tile is put into its stage there, and the one two further on loaded if there is one (`more`).
    auto half_step = [&](auto set_tag, int s0, bool fixed, bool reads, bool loads, int to, bool more_loads) {
      constexpr int set = decltype(set_tag)::value;
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        acc[q >> 2][q & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][q & 3], fa[set][q >> 2], acc[q >> 2][q & 3], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if ((q & 1) == 0 && reads) read_one(set ^ 1, q >> 1, s0, fixed);
        if ((q & 3) == 1 && loads) {
          put_one(set, q >> 2, to);
          if (!STAGED || more_loads) issue_one(set, q >> 2, to);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto clear_beyond = [&](int h) {            // in fragments of half h of the last step, in BOTH operands: the padding may hold anything
      if (left_adding == 0) return;
      const int valid = left_adding - h * kMfmaBK - (lane >> 4) * 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        fa[h][i] = __builtin_bit_cast(bf16x8_t, mask_tail8(__builtin_bit_cast(u32x4_t, fa[h][i]), valid));
        fb[h][i] = __builtin_bit_cast(bf16x8_t, mask_tail8(__builtin_bit_cast(u32x4_t, fb[h][i]), valid));
      }
    };
    // (the compiler moves no LDS access across it)
    auto barrier = [&]() {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    // waits until all but the `after` tiles loaded last have landed (and this wave's fragment reads are over)
    auto landed = [&](int after) {
      if (after >= 4) __builtin_amdgcn_s_waitcnt(waitcnt_imm(16, 0));
      else if (after >= 3) __builtin_amdgcn_s_waitcnt(waitcnt_imm(12, 0));
      else if (after >= 2) __builtin_amdgcn_s_waitcnt(waitcnt_imm(8, 0));
      else if (after >= 1) __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 0));
      else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
      barrier();
    };
    if (tiles > 0) {
      const std::integral_constant<int, 0> even{};
      const std::integral_constant<int, 1> odd{};
      for (int s = 0; s < min(tiles, L); s += 2) {
        if (masked && to_load == 1) place_last();
#pragma unroll
        for (int i = 0; i < 8; ++i) issue_one(i >> 2, i & 3, s + (i >> 2));
        if constexpr (STAGED)
#pragma unroll
          for (int i = 0; i < 8; ++i) put_one(i >> 2, i & 3, s + (i >> 2));
      }
      if (STAGED && L < tiles)
#pragma unroll
        for (int i = 0; i < 8; ++i) issue_one(i >> 2, i & 3, 0);
      if (STAGED) __syncthreads();
      else landed(min(tiles, L) - 2);
#pragma unroll
      for (int i = 0; i < 8; ++i) read_one(0, i, 0, true);
      const int full = tiles - L;               // tiles below this one load another while they are multiplied
      // waits until the next step's two tiles are there and this one's fragment reads are over, `after` later tiles being on their way
      auto arrive = [&](int after) {
        if (STAGED) {
          __builtin_amdgcn_s_waitcnt(waitcnt_lgkm(0));
          barrier();
        } else {
          landed(after);
        }
      };
      int k = 0;                                // tile in fragment set 0
      auto step = [&](auto u_tag) {             // a K step whose tiles are in stages 2 u and 2 u + 1 (modulo R)
        constexpr int s0 = 2 * decltype(u_tag)::value % R, next = (s0 + 2) % R, to = (s0 + L) % R;
        half_step(even, s0, true, true, true, to, true);
        if constexpr (STAGED) {
          arrive(0);
        } else {                                // both tiles of the next step have landed, L - 3 later ones are on their way
          __builtin_amdgcn_s_waitcnt(kReadsDone ? waitcnt_imm(4 * (L - 3), 0) : waitcnt_vm(4 * (L - 3)));
          barrier();
        }
        half_step(odd, next, true, true, true, (to + 1) % R, true);
        step_done();
        k += 2;
      };
      const int unrolled = STAGED || masked ? (run_on ? 0 : full - 2) : full;      // (a step whose loads or fragments are special is not among these)
      for (; k + 2 * kMidUnroll <= unrolled; ) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
        step(std::integral_constant<int, 4>{});
      }
      int s0 = 0, to = L;                       // the rest with stages that are worked out
      auto follow = [](int s, int by) { return s + by >= R ? s + by - R : s + by; };
      for (; k < full; k += 2) {
        const bool more_loads = k + 2 < full;
        if (masked && to_load == 1) place_last();
        if (masked && to_add == 1) clear_beyond(0);
        half_step(even, s0, false, true, true, to, more_loads);
        s0 = follow(s0, 2);
        arrive(L - 3);
        if (masked && to_add == 1) clear_beyond(1);
        half_step(odd, s0, false, true, true, follow(to, 1), more_loads);
        step_done();
        to = follow(to, 2);
      }
      for (; k + 2 < tiles; k += 2) {           // everything is loaded
        if (masked && to_add == 1) clear_beyond(0);
        half_step(even, s0, false, true, false, 0, false);
        s0 = follow(s0, 2);
        arrive(tiles - k - 4);
        if (masked && to_add == 1) clear_beyond(1);
        half_step(odd, s0, false, true, false, 0, false);
        step_done();
      }
      if (masked) clear_beyond(0);
      half_step(even, s0, false, true, false, 0, false);
      if (masked) clear_beyond(1);
      half_step(odd, s0, false, false, false, 0, false);
      step_done();
    }
    if (!masked && left > 0) {                  // a tile that may be partial, through registers, and a whole one before it if there are two
      typedef GSPMD_GLOBAL const unsigned char* gbytes;
      const int at_part = left > kMfmaBK ? 1 : 0, here = left - at_part * kMfmaBK;
      const bf16_bits *a_tail = a_base + tiles * a_tile, *b_tail = b_base + tiles * b_tile;
      int lane_rest = lane_here();              // (the places are worked out here, not kept in registers through the loop above)
      asm volatile("" : "+v"(lane_rest));
      const int lane_of = kFewRegisters ? lane_rest : lane;
      auto a_place = [&](int j) { return AKM ? a_off[0][j] : kc_load_offset(wave * 2 + j, lane_rest, m0, P.Mv, P.lda); };
      auto b_place = [&](int j) { return BKC ? kc_load_offset(wave * 2 + j, lane_rest, n0, P.Nv, P.ldb) : b_off[0][j]; };
      auto chunk = [&](bool kmajor, const bf16_bits* base, int off, int q, int valid) -> u32x4_t {
        u32x4_t v = {0u, 0u, 0u, 0u};
        const int kr = kmajor ? q * 4 + (lane_of >> 4) : ((lane_of & 3) ^ swz_a(q * 16 + (lane_of >> 2))) * 8;
        if (!kmajor) v = STAGED ? load_k_elements((GSPMD_GLOBAL const uint16_t*)((gbytes)base + off), valid - kr) : load_k_chunk((GSPMD_GLOBAL const uint32_t*)((gbytes)base + off), valid - kr);
        else if (kr < valid) v = *(GSPMD_GLOBAL const u32x4_elements_t*)((gbytes)base + off);
        return v;
      };
      auto load = [&](int tile, int valid, u32x4_t (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          v[j] = chunk(AKM, a_tail + tile * a_tile, a_place(j), wave * 2 + j, valid);
          v[2 + j] = chunk(!BKC, b_tail + tile * b_tile, b_place(j), wave * 2 + j, valid);
        }
      };
      auto put = [&](int tile, const u32x4_t (&v)[4]) {
        unsigned char* at = smem + tile * kMidStage + wave * 2048 + lane_of * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4_t*>(at + (i >> 1) * kMidPart + (i & 1) * 1024) = v[i];
      };
      u32x4_t part[4], whole[4];
      load(at_part, here, part);
      if (STAGED && at_part) load(0, kMfmaBK, whole);
      __syncthreads();                          // every wave has read the tiles before
      if (at_part) {
        if constexpr (STAGED) {
          put(0, whole);
        } else {
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            global_to_lds16(a_tail, a_place(j), lds_wave + j * 1024);
            global_to_lds16(b_tail, b_place(j), lds_wave + kMidPart + j * 1024);
          }
        }
      }
      put(at_part, part);
      if (!STAGED && at_part) __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
      __syncthreads();
      for (int tile = 0; tile <= at_part; ++tile) {
        const uint32_t stage = tile * kMidStage;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          fb[0][i] = BKC ? read_kc(lds0 + stage + kMidPart + kc_frag_offset(wn, lane_of) + i * 1024) : read_km(b_reg[0][BKC ? 0 : i] + stage);
          fa[0][i] = AKM ? read_km(a_reg[0][AKM ? i : 0] + stage) : read_kc(lds0 + stage + kc_frag_offset(wm, lane_of) + i * 1024);
        }
        multiply(0);
      }
    }
    if (!run_on) add_member(member == 0);
  }

  // ---- epilogue
  GSPMD_GLOBAL TOut* const C = (GSPMD_GLOBAL TOut*)P.C;
  constexpr int kAtOnce = sizeof(TOut) == 2 ? 4 : 2;
  static_assert(4 * line_slice<TOut>(kAtOnce) <= R * kMidStage, "");
  constexpr bool kHinted = !STAGED && sizeof(TOut) == 2;
  const int lane_end = lane_here(), t_end = kFewRegisters ? wave * 64 + lane_end : t;
  __syncthreads();                              // every wave's fragment reads are over
  store_lines<TOut, 4, kAtOnce, kHinted ? kLinesThrough : kLinesPlain>(smem + wave * line_slice<TOut>(kAtOnce), C, P, m0 + wm, n0 + wn, m0 + kMidTile <= P.Mv && n0 + kMidTile <= P.Nv, kHinted ? epilogue & ~kStorePast : epilogue, lane_end, [&](int i, int j) {
    if constexpr (CHAIN) return sum[i][j]; else return acc[i][j];
  }, kHinted && (epilogue & kStorePast) != 0);
  // zeros of the static block below the last row tile, over this tile's columns (what lies further down, and whole tile
  // columns of padding, the fill kernel clears)
  const int m_done = min(m_nom + kMidTile, P.Mv), moved_end = n0 + kMidTile, col_end = min(n_nom + kMidTile, P.Ns);
  if (n0 < n_nom) zero_block<kMidThreads, TOut>(C, P.ldc, m0, m_done, moved_end, col_end, t_end);            // right of a tile that was moved back
  if (m_done == P.Mv) {
    zero_block<kMidThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), n0, min(moved_end, P.Ns), t_end);
    if (n0 < n_nom) zero_block<kMidThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), moved_end, col_end, t_end);
  }
}

template <typename TOut, int LAYOUT, bool CHAIN, int PER_CU, bool STAGED = false>
inline bool launch_dot_mid_as(const MfmaLaunch& l, hipStream_t stream) {
  constexpr int lds = mid_stages<PER_CU>() * kMidStage;
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::call_once(once[dev], [dev] {
    ok[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&dot_mid_kernel<TOut, LAYOUT, CHAIN, PER_CU, STAGED>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
  });
  if (!ok[dev]) return false;
  hipLaunchKernelGGL((dot_mid_kernel<TOut, LAYOUT, CHAIN, PER_CU, STAGED>), dim3(static_cast<unsigned>(l.tiles)), dim3(kMidThreads), lds, stream, *l.inl, l.tab,
                     l.n_prob, !STAGED && sizeof(TOut) == 2 && l.past ? l.epilogue | kStorePast : l.epilogue);
  return hipGetLastError() == hipSuccess;
}

template <int LAYOUT, bool CHAIN>
bool launch_dot_mid_out(const MfmaLaunch& l, int32_t out_dtype, hipStream_t stream) {
  if (l.tiles <= kMidAlone)
    return out_dtype == GSPMD_F32 ? launch_dot_mid_as<float, LAYOUT, CHAIN, 1>(l, stream) : launch_dot_mid_as<bf16_bits, LAYOUT, CHAIN, 1>(l, stream);
  return out_dtype == GSPMD_F32 ? launch_dot_mid_as<float, LAYOUT, CHAIN, 2>(l, stream) : launch_dot_mid_as<bf16_bits, LAYOUT, CHAIN, 2>(l, stream);
}

template <int LAYOUT>
bool launch_dot_mid_layout(const MfmaLaunch& l, int32_t out_dtype, bool chain, bool staged, hipStream_t stream) {
  if (staged)
    return out_dtype == GSPMD_F32 ? launch_dot_mid_as<float, LAYOUT, false, 2, true>(l, stream) : launch_dot_mid_as<bf16_bits, LAYOUT, false, 2, true>(l, stream);
  return chain ? launch_dot_mid_out<LAYOUT, true>(l, out_dtype, stream) : launch_dot_mid_out<LAYOUT, false>(l, out_dtype, stream);
}

}  // namespace gspmd
