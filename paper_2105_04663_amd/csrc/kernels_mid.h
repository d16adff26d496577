// bf16 MFMA contraction in 128 x 128 tiles, two workgroups per compute unit: for launches that 256 x 256 tiles (one
// workgroup per compute unit, 9 us beside its K loop) leave waiting or idle -- few output tiles, short K -- and for sums over
// a contracting mesh dimension, which it forms without a workspace: a workgroup takes the members' K ranges one after
// the other and adds each member's finished product to a second set of accumulators, so the sum is ((p0 + p1) + p2) + ..
// in fp32 as everywhere else.  Products take their 32-wide K tiles in the order and with the instruction of
// dot_mfma_kernel: results are bit-identical to it.  16-byte aligned operands only.
//
// What bounds it: what a compute unit draws from L2, 16 KiB per 32-wide K tile for 256 cycles of the matrix cores.  With two
// workgroups on each (2048 x 2048 x 4096) its L1 keeps about 91 lines of 128 bytes in flight, 322 cycles each, and stalls on them
// for 45 % of the cycles; matrix cores busy for 42 %, LDS for 21 %.  (One workgroup, 2048 x 2048 x 2048: 32 % and 16 %.)
// Five LDS stages of a 32-wide K tile (80 KiB) filled by direct global->LDS loads, up to five tiles ahead, one barrier per
// tile; a wave reads the next tile's fragments while it multiplies this one's.
// A K-major operand lies in its stage as [32 k][128], read with the transpose read; a K-contiguous one as [128][32 k].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "kernels_basic.h"
#include "launch.h"
#include "mfma_common.h"
#include "plan.h"
#include "tile_index.h"

namespace gspmd {

constexpr int kMidPart = kMidTile * kMfmaBK * 2;      // 8 KiB: one operand's 32-wide K tile
constexpr int kMidStage = 2 * kMidPart, kMidStages = 5;
constexpr int kMidLds = kMidStages * kMidStage;

// K-major part [32 k][128 columns]: 16 chunks of 16 bytes per k row.  Chunk pairs (one 16-column block) are XOR-swizzled by
// the row, so that the 4 rows x 32 bytes that a 16-lane group reads and those of the group beside it (8 rows further)
// lie in different banks.
__device__ __forceinline__ int mid_swz(int krow) { return ((krow & 3) | (((krow >> 3) & 1) << 2)) << 1; }
// load instruction q (0..7) of a K-major part: k rows 4 q .. 4 q + 3, 16 lanes per row; chunks past the valid extent reuse
// the last valid chunk
__device__ __forceinline__ int mid_km_load_offset(int q, int lane, int c0, int cols_valid, int ld) {
  const int kr = q * 4 + (lane >> 4);
  int n = c0 + (((lane & 15) ^ mid_swz(kr)) << 3);
  if (n >= cols_valid) n = ((cols_valid - 1) >> 3) << 3;
  return (kr * ld + (n - c0)) * 2;
}
// fragment of the 16-column block at `base` (block b further at ^ (b << 5) for a base that is a multiple of 64)
__device__ __forceinline__ int mid_km_frag_offset(int base, int lane) {
  const int i = lane & 15, krow = (lane >> 4) * 8 + (i >> 2), cl = base + (i & 3) * 4;
  return krow * 256 + (((cl >> 3) ^ mid_swz(krow)) << 4) + (cl & 7) * 2;
}

template <typename TOut, int LAYOUT, bool CHAIN>
__global__ __launch_bounds__(kMidThreads, 2) void dot_mid_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
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
  const int m0 = (band * kBandRows + in_band % rows_in_band) * kMidTile, n0 = (in_band / rows_in_band) * kMidTile;
  const int members = CHAIN ? max(P.join_count, 1) : 1;

  float4_t acc[4][4], sum[CHAIN ? 4 : 1][CHAIN ? 4 : 1];
  const int a_frag = AKM ? mid_km_frag_offset(wm, lane) : kc_frag_offset(wm, lane);
  const int b_frag = kMidPart + (BKC ? kc_frag_offset(wn, lane) : mid_km_frag_offset(wn, lane));
  auto read_kc = [&](const unsigned char* p) { return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(p)); };
  auto read_km = [&](const unsigned char* p) {
    short8_t both;
    both.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(p));
    both.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_t*)(p + 4 * 256));
    return __builtin_bit_cast(bf16x8_t, both);
  };
  bf16x8_t fa[2][4], fb[2][4];                  // fragments of two tiles: one being multiplied, the next being read
  auto read_frags = [&](int stage, int set) {
    const unsigned char* base = smem + stage * kMidStage;
#pragma unroll
    for (int i = 0; i < 4; ++i) fb[set][i] = BKC ? read_kc(base + b_frag + i * 1024) : read_km(base + (b_frag ^ (i << 5)));
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[set][i] = AKM ? read_km(base + (a_frag ^ (i << 5))) : read_kc(base + a_frag + i * 1024);
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
  };

  for (int member = 0; member < members; ++member) {
    if (CHAIN && member > 0) {
      P = problem_at(tab, which + member);
      __syncthreads();                          // every wave has read the last tile of the member before
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    const bf16_bits* a_base = static_cast<const bf16_bits*>(P.A) + (AKM ? static_cast<int64_t>(m0) : static_cast<int64_t>(m0) * P.lda);
    const bf16_bits* b_base = static_cast<const bf16_bits*>(P.B) + (BKC ? static_cast<int64_t>(n0) * P.ldb : static_cast<int64_t>(n0));
    const int64_t a_tile = AKM ? static_cast<int64_t>(kMfmaBK) * P.lda : kMfmaBK, b_tile = BKC ? kMfmaBK : static_cast<int64_t>(kMfmaBK) * P.ldb;
    const int tiles = P.Kv / kMfmaBK, left = P.Kv - tiles * kMfmaBK;
    int a_off[2], b_off[2];                     // this wave's two load instructions of each operand's part
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = wave * 2 + j;
      a_off[j] = AKM ? mid_km_load_offset(q, lane, m0, P.Mv, P.lda) : kc_load_offset(q, lane, m0, P.Mv, P.lda);
      b_off[j] = BKC ? kc_load_offset(q, lane, n0, P.Nv, P.ldb) : mid_km_load_offset(q, lane, n0, P.Nv, P.ldb);
    }
    const bf16_bits *a_next = a_base, *b_next = b_base;
    int fill = 0;                               // stage the next load goes to
    auto issue = [&]() {
      const uint32_t at = lds0 + fill * kMidStage + wave * 2048;
#pragma unroll
      for (int j = 0; j < 2; ++j) global_to_lds16(a_next, a_off[j], at + j * 1024);
#pragma unroll
      for (int j = 0; j < 2; ++j) global_to_lds16(b_next, b_off[j], at + kMidPart + j * 1024);
      a_next += a_tile;
      b_next += b_tile;
      fill = fill == kMidStages - 1 ? 0 : fill + 1;
    };
    for (int s = 0; s < min(tiles, kMidStages); ++s) issue();
    int stage = 0;                              // of the tile whose fragments are read next
    auto next_stage = [&]() { stage = stage == kMidStages - 1 ? 0 : stage + 1; };
    // Waits until the tile to be read has landed, `after` later tiles being in flight, and every wave has its fragments of
    // the tile before in registers (lgkmcnt 0): that tile's stage is free.
    auto arrive = [&](int after) {
      if (after >= 4) __builtin_amdgcn_s_waitcnt(waitcnt_imm(16, 0));
      else if (after == 3) __builtin_amdgcn_s_waitcnt(waitcnt_imm(12, 0));
      else if (after == 2) __builtin_amdgcn_s_waitcnt(waitcnt_imm(8, 0));
      else if (after == 1) __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 0));
      else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
      __builtin_amdgcn_s_barrier();
    };
    if (tiles > 0) {
      arrive(min(tiles, kMidStages) - 1);
      read_frags(0, 0);
      next_stage();
      int k = 0;                                // tile in fragment set 0
      for (; k + kMidStages + 2 <= tiles; k += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          __builtin_amdgcn_s_waitcnt(waitcnt_imm(12, 0));        // tile k + h + 1 is there; k + h + 2 .. k + h + 4 on their way
          __builtin_amdgcn_s_barrier();
          issue();                                               // tile k + h + 5 into the stage of tile k + h
          read_frags(stage, h ^ 1);
          next_stage();
          __builtin_amdgcn_sched_barrier(0);                     // the reads are under way before the MFMAs, and those do not
          multiply(h);                                           // move behind the next wait
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      for (; k < tiles; k += 2) {               // at most six tiles left, one of them still to be loaded
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (k + h >= tiles) break;
          if (k + h + 1 < tiles) {
            const int loaded = min(tiles, k + h + kMidStages);   // tiles whose loads have been issued
            arrive(loaded - (k + h + 2));
            if (loaded < tiles) issue();
            read_frags(stage, h ^ 1);
            next_stage();
          }
          multiply(h);
        }
      }
    }
    if (left > 0) {                             // the partial tile, through registers: zeros beyond the valid K in BOTH operands
      typedef GSPMD_GLOBAL const unsigned char* gbytes;
      u32x4_t ta[2], tb[2];
      auto chunk = [&](bool kmajor, const bf16_bits* base, int off, int q) -> u32x4_t {
        u32x4_t v = {0u, 0u, 0u, 0u};
        const int kr = kmajor ? q * 4 + (lane >> 4) : ((lane & 3) ^ swz_a(q * 16 + (lane >> 2))) * 8;
        if (kr < left) {
          v = *(GSPMD_GLOBAL const u32x4_t*)((gbytes)base + off);
          if (!kmajor && kr + 8 > left) v = mask_tail8(v, left - kr);
        }
        return v;
      };
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        ta[j] = chunk(AKM, a_base + tiles * a_tile, a_off[j], wave * 2 + j);
        tb[j] = chunk(!BKC, b_base + tiles * b_tile, b_off[j], wave * 2 + j);
      }
      __syncthreads();                          // every wave has read the last whole tile
      unsigned char* at = smem + wave * 2048 + lane * 16;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        *reinterpret_cast<u32x4_t*>(at + j * 1024) = ta[j];
        *reinterpret_cast<u32x4_t*>(at + kMidPart + j * 1024) = tb[j];
      }
      __syncthreads();
      read_frags(0, 0);
      multiply(0);
    }
    if constexpr (CHAIN) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[i][j] = member == 0 ? acc[i][j] : sum[i][j] + acc[i][j];
    }
  }

  // ---- epilogue: a lane holds columns n .. n + 3 of row m per 16 x 16 block
  GSPMD_GLOBAL TOut* const C = (GSPMD_GLOBAL TOut*)P.C;
  typedef TOut out4 __attribute__((ext_vector_type(4), aligned(sizeof(TOut))));
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
  const bool inside = m0 + kMidTile <= P.Mv && n0 + kMidTile <= P.Nv;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + wm + i * 16 + (lane & 15);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + wn + j * 16 + (lane >> 4) * 4;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float x;
        if constexpr (CHAIN) x = sum[i][j][e]; else x = acc[i][j][e];
        v[e] = apply_epilogue(x, epilogue);
      }
      if (!inside) {
        if (m >= P.Mv || n >= P.Ns) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e) if (n + e >= P.Nv) v[e] = 0.f;
      }
      out4 o;
      if constexpr (sizeof(TOut) == 2) {
        const bf16x4_t h = {static_cast<__bf16>(v[0]), static_cast<__bf16>(v[1]), static_cast<__bf16>(v[2]), static_cast<__bf16>(v[3])};
        o = __builtin_bit_cast(out4, h);
      } else {
        o = out4{v[0], v[1], v[2], v[3]};
      }
      GSPMD_GLOBAL TOut* c = C + static_cast<int64_t>(m) * P.ldc + n;
      if (inside || n + 4 <= P.Ns) *(GSPMD_GLOBAL out4*)c = o;
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) if (n + e < P.Ns) c[e] = o[e];
    }
  }
  // zeros of the static block below the last row tile, over this tile's columns (what lies further down, and whole tile
  // columns of padding, the fill kernel clears)
  if (m0 + kMidTile >= P.Mv)
    zero_block<kMidThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), n0, min(n0 + kMidTile, P.Ns), t);
}

template <typename TOut, int LAYOUT, bool CHAIN>
inline bool launch_dot_mid_as(const MfmaLaunch& l, hipStream_t stream) {
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::call_once(once[dev], [dev] {
    ok[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&dot_mid_kernel<TOut, LAYOUT, CHAIN>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, kMidLds) == hipSuccess;
  });
  if (!ok[dev]) return false;
  hipLaunchKernelGGL((dot_mid_kernel<TOut, LAYOUT, CHAIN>), dim3(static_cast<unsigned>(l.tiles)), dim3(kMidThreads), kMidLds, stream, *l.inl, l.tab,
                     l.n_prob, l.epilogue);
  return hipGetLastError() == hipSuccess;
}

template <int LAYOUT>
bool launch_dot_mid_layout(const MfmaLaunch& l, int32_t out_dtype, bool chain, hipStream_t stream) {
  if (out_dtype == GSPMD_F32) return chain ? launch_dot_mid_as<float, LAYOUT, true>(l, stream) : launch_dot_mid_as<float, LAYOUT, false>(l, stream);
  return chain ? launch_dot_mid_as<bf16_bits, LAYOUT, true>(l, stream) : launch_dot_mid_as<bf16_bits, LAYOUT, false>(l, stream);
}

}  // namespace gspmd
