// float32 contraction on the matrix cores: C[m,n] = sum_k A[m,k] * B[k,n], every product and sum in float32
// (v_mfma_f32_16x16x4_f32), operands in any of the four layouts, at any alignment.
//
// Matrix-core bound: 256 flop per clock and compute unit, a sixteenth of the bf16 rate, so one 64 x 64 tile per workgroup
// feeds the cores from L2 at 16 bytes per clock, and small tiles are what keeps all compute units equally busy (2048 x
// 2048 x 3000 on 8 partitions: 1536 tiles, six per compute unit).  Four waves of 32 x 32.
//
// What the matrix cores lose they lose to vector instructions between the MFMAs, however many workgroups are resident: an address
// worked out per load and per LDS read (12 instructions beside 32 MFMAs) costs 13 % (2048 x 2048 x 3000: 201 us, now 180; 4096^3: 1060, 916).
// So the loop has none: 16-byte loads go straight into LDS from bases in scalar registers and constant offsets of a lane, and the stages come round
// in unrolled code, so that LDS addresses are constants.  K in steps of 32 through three stages (two where four workgroups share a
// compute unit), one barrier per step; the reads of the next 16 k's fragments and the loads of the step three further on are issued one at a
// time between the MFMAs, so that a workgroup that is left alone on a compute unit keeps its matrix cores busy too.
// A lane's four k of a K-contiguous fragment are one 16-byte LDS read; the four MFMAs that use them take k = 4 g + i of every 16 (g =
// lane / 16), for both operands alike, which only reorders the sum.
// Measured (us; operands through registers and ds_write, reads ahead of a step's MFMAs / now): 2048 x 2048 x 3000 on a 2 x 4 mesh 230 / 180 (140
// TFLOP/s), 4096^3 1097 / 916 (150; 155 is what the cores reach without memory), 2048^3 144 / 118, 1024 x 4096 x 1024 86 / 62, 94 x 1790 x 491 on a 2 x 4 mesh 43 / 31.
// Matrix cores busy for 96 % of a compute unit's cycles at 2048 x 2048 x 3000 (81 before), LDS 4, no bank conflicts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels_basic.h"
#include "mfma_common.h"
#include "plan.h"
#include "tile_index.h"

namespace gspmd {

constexpr int kF32Tile = 64, kF32BK = 32, kF32Threads = 256;
constexpr int kF32MaxStride = 1 << 27;                  // elements: a load instruction's rows stay within 32-bit offsets (of bytes)
constexpr int kF32Part = kF32Tile * kF32BK * 4;        // 8 KiB: one operand's share of a K step
template <bool LEAN> constexpr int f32_stages() { return LEAN ? 2 : 3; }

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// LEAN: LDS for four workgroups on a compute unit (f32_four).  WIDE: rows beyond 32-bit offsets (512 MiB and more), a lane's offsets in 64 bits and one
// addition per load.
template <int LAYOUT, bool LEAN, bool WIDE = false>
__global__ __launch_bounds__(kF32Threads, LEAN ? 4 : 3) void dot_f32_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
  constexpr int R = f32_stages<LEAN>();
  __shared__ __attribute__((aligned(1024))) unsigned char lds[R * 2 * kF32Part];        // [stage][operand]
  typedef GSPMD_GLOBAL const float* gfloats;
  typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
  typedef __attribute__((address_space(3))) const float lds_float;
  const int t = threadIdx.x, lane = t & 63, group = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  const int tile = logical_tile(blockIdx.x, gridDim.x);
  const Problem P = lookup_problem(tab, n_prob, tile);
  const int local = tile - P.tile_begin;
  // bands of 8 tile rows, the row index running fastest: tiles that are in flight together share operand panels in L2
  const int tiles_m = (P.Mv + kF32Tile - 1) / kF32Tile;
  const int band = local / (8 * P.tiles_n), in_band = local - band * 8 * P.tiles_n, rows_in_band = min(8, tiles_m - band * 8);
  const int m0 = (band * 8 + in_band % rows_in_band) * kF32Tile, n0 = (in_band / rows_in_band) * kF32Tile;

  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const gfloats A = (gfloats)P.A, B = (gfloats)P.B;
  // Where the j-th of its wave's two loads of an operand's part begins at K step 0: a base in scalar registers, which moves on from step to step, and
  // this lane's offset.  An index along m or n beyond the valid extent becomes the last valid row (K-contiguous) or the last four columns
  // (K-major): those results are not stored.  A K-major chunk that straddles the end is the last four columns as well; its columns' readers
  // find them there (f32_km_column).
  auto load_base = [&](bool kmajor, gfloats base, int64_t ld, int x0, int valid, int j) {
    const int q = wave * 2 + j;
    return reinterpret_cast<uint64_t>(base + (kmajor ? q * 4 : min(x0 + q * 8, valid - 1)) * ld);
  };
  typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type offset_t;
  auto load_offset = [&](bool kmajor, int64_t ld, int x0, int valid, int j) -> offset_t {
    const int q = wave * 2 + j, row = x0 + q * 8;
    if (kmajor) return static_cast<offset_t>((lane >> 4) * ld + f32_km_first(x0 + f32_km_chunk(q, lane) * 4, valid)) * 4;
    return static_cast<offset_t>((min(row + (lane >> 3), valid - 1) - min(row, valid - 1)) * ld + f32_kc_chunk(q, lane) * 4) * 4;
  };
  uint64_t a_at[2], b_at[2];
  offset_t a_off[2], b_off[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    a_at[j] = load_base(AKM, A, P.lda, m0, P.Mv, j);
    b_at[j] = load_base(!BKC, B, P.ldb, n0, P.Nv, j);
    a_off[j] = load_offset(AKM, P.lda, m0, P.Mv, j);
    b_off[j] = load_offset(!BKC, P.ldb, n0, P.Nv, j);
  }
  // no whole chunk along m or n (or rows that this variant's offsets do not reach, which the host gives to WIDE)
  const bool slow = (AKM && P.Mv < 4) || (!BKC && P.Nv < 4) || (!WIDE && max(P.lda, P.ldb) >= kF32MaxStride);
  const int64_t a_step = (AKM ? static_cast<int64_t>(P.lda) * kF32BK : kF32BK) * 4, b_step = (BKC ? kF32BK : static_cast<int64_t>(P.ldb) * kF32BK) * 4;
  // the i-th of this wave's four loads of the next K step
  auto load_one = [&](int i, uint32_t stage_at) {
    const uint32_t to = stage_at + (i >> 1) * kF32Part + (wave * 2 + (i & 1)) * 1024;
    auto load = [&](uint64_t from, offset_t off) {
      if constexpr (WIDE) global_to_lds16(from + off, to);
      else global_to_lds16(reinterpret_cast<const void*>(from), off, to);
    };
    if (i < 2) {
      load(a_at[i & 1], a_off[i & 1]);
      a_at[i & 1] += a_step;
    } else {
      load(b_at[i & 1], b_off[i & 1]);
      b_at[i & 1] += b_step;
    }
  };
  // Where this lane's fragments are in an operand's part: K-contiguous, four k of a row in one read (halves of the step 64 bytes apart by
  // XOR); K-major, one column of each of two 16-column blocks.
  uint32_t a_from[2], b_from[2];
  auto place = [&](bool shifted) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int x = wm + 16 * i + (lane & 15), y = wn + 16 * i + (lane & 15);
      a_from[i] = lds0 + (AKM ? f32_km_place(shifted ? f32_km_column(x, P.Mv - m0) : x, group) : f32_kc_place(wm + (lane & 15), group) ^ (i * 64));
      b_from[i] = lds0 + kF32Part + (!BKC ? f32_km_place(shifted ? f32_km_column(y, P.Nv - n0) : y, group) : f32_kc_place(wn + (lane & 15), group) ^ (i * 64));
    }
  };
  place(true);
  f32x4 fa[2][2], fb[2][2];                     // fragments of two 16-wide halves: one being multiplied, the next being read
  // fragment i (lhs 0, 1, rhs 0, 1) of half h of the step whose stage is at `stage_at` (from the first one)
  auto read_one = [&](int h, int i, uint32_t stage_at) {
    auto four = [&](bool kmajor, const uint32_t (&from)[2], int b) -> f32x4 {
      if (!kmajor) return *(lds_f32x4*)(uintptr_t)(stage_at + from[h] + b * 16 * 128);
      f32x4 v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = *(lds_float*)(uintptr_t)(stage_at + from[b] + (h * 16 + q) * 256);
      return v;
    };
    if (i < 2) fa[h][i] = four(AKM, a_from, i);
    else fb[h][i & 1] = four(!BKC, b_from, i & 1);
  };
  // Half a step: sixteen MFMAs, and between them the reads of the next half's fragments and the loads of a step further on.
  auto half_step = [&](auto half, bool reads, uint32_t read_at, bool loads, uint32_t load_at) {
    constexpr int h = decltype(half)::value;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = (q >> 1) & 1, j = q & 1;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[h][j][q >> 2], fa[h][i][q >> 2], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (reads && (q & 1) == 0 && q < 8) read_one(h ^ 1, q >> 1, read_at);
      if (loads && q % 3 == 2 && q < 12) load_one(q / 3, load_at);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const std::integral_constant<int, 0> first{};
  const std::integral_constant<int, 1> second{};
  auto barrier = [&]() {                        // (the compiler moves no LDS access across it)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // waits until all but the `after` steps loaded last have landed, and this wave's fragment reads are over
  auto landed = [&](int after) {
    if (after >= 2) __builtin_amdgcn_s_waitcnt(waitcnt_imm(8, 0));
    else if (after == 1) __builtin_amdgcn_s_waitcnt(waitcnt_imm(4, 0));
    else __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));
    barrier();
  };

  const int whole = slow ? 0 : P.Kv / kF32BK;
  if (whole > 0) {
    constexpr uint32_t kStage = 2 * kF32Part;
    for (int s = 0; s < min(whole, R); ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) load_one(i, lds0 + s * kStage);
    landed(min(whole, R) - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) read_one(0, i, 0);
    int s = 0;
    // a step's stage is free when its second half's fragments are read, before that half is multiplied
    auto step = [&](uint32_t here, uint32_t next) {
      half_step(first, true, here, false, 0);
      landed(R - 2);
      half_step(second, true, next, true, lds0 + here);
    };
    for (; s + 2 * R <= whole; s += R)          // the stages are constants of the code
#pragma unroll
      for (int u = 0; u < R; ++u) step(u * kStage, (u + 1) % R * kStage);
    uint32_t here = 0;                          // the stage of step s
    auto after = [&](uint32_t at) { return at == (R - 1) * kStage ? 0 : at + kStage; };
    for (; s + R < whole; ++s) {
      step(here, after(here));
      here = after(here);
    }
    for (; s + 1 < whole; ++s) {                // everything is loaded
      half_step(first, true, here, false, 0);
      landed(min(whole - s, R) - 2);
      half_step(second, true, after(here), false, 0);
      here = after(here);
    }
    half_step(first, true, here, false, 0);
    half_step(second, false, 0, false, 0);
  }
  if (whole * kF32BK < P.Kv) {                  // what is left of K, or an extent below a chunk: element by element, zeros beyond in BOTH operands
    place(false);
    for (int k0 = whole * kF32BK; k0 < P.Kv; k0 += kF32BK) {
      auto fetch = [&](bool kmajor, gfloats base, int64_t ld, int x0, int valid, int j) -> f32x4 {
        const int q = wave * 2 + j;
        const int x = x0 + (kmajor ? f32_km_chunk(q, lane) * 4 : q * 8 + (lane >> 3)), k = k0 + (kmajor ? q * 4 + (lane >> 4) : f32_kc_chunk(q, lane) * 4);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int xe = kmajor ? x + e : x, ke = kmajor ? k : k + e;
          if (xe < valid && ke < P.Kv) v[e] = base[kmajor ? ke * ld + xe : xe * ld + ke];
        }
        return v;
      };
      f32x4 v[4];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        v[j] = fetch(AKM, A, P.lda, m0, P.Mv, j);
        v[2 + j] = fetch(!BKC, B, P.ldb, n0, P.Nv, j);
      }
      __syncthreads();                          // every wave has read the step before
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(lds + (i >> 1) * kF32Part + (wave * 2 + (i & 1)) * 1024 + lane * 16) = v[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) read_one(i >> 2, i & 3, 0);
      half_step(first, false, 0, false, 0);
      half_step(second, false, 0, false, 0);
    }
  }

  // a lane holds four consecutive columns of a row per 16 x 16 block; the static block's part of this tile is written
  // whole, zeros outside the valid extents
  GSPMD_GLOBAL float* const C = (GSPMD_GLOBAL float*)P.C;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + wm + 16 * i + (lane & 15);
    if (m >= P.Ms) continue;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn + 16 * j + (lane >> 4) * 4;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (m < P.Mv && n + e < P.Nv) ? apply_epilogue(acc[i][j][e], epilogue) : 0.f;
      GSPMD_GLOBAL float* c = C + static_cast<int64_t>(m) * P.ldc + n;
      if (n + 4 <= P.Ns) *(GSPMD_GLOBAL f32x4_any*)c = o;
      else
#pragma unroll
        for (int e = 0; e < 4; ++e) if (n + e < P.Ns) c[e] = o[e];
    }
  }
}

}  // namespace gspmd
