// float32 contraction on the matrix cores: C[m,n] = sum_k A[m,k] * B[k,n], every product and sum in float32
// (v_mfma_f32_16x16x4_f32), operands in any of the four layouts, at any alignment.
//
// Matrix-core bound: 256 flop per clock and compute unit, a sixteenth of the bf16 rate, so one 64 x 64 tile per workgroup
// feeds the cores from L2 at 16 bytes per clock, and small tiles are what keeps all compute units equally busy (2048 x
// 2048 x 3000 on 8 partitions: 1536 tiles, six per compute unit).  Four waves of 32 x 32; K in steps of 32 through two
// LDS buffers, loads two steps ahead, one barrier per step, three workgroups on a compute unit, or four where that shares its tiles out
// better (f32_four).  128-row tiles, three on a compute unit, need more registers than there are: 275 us below.  A lane's four k of a K-contiguous fragment are one 16-byte LDS read; the four MFMAs
// that use them take k = 4 g + i of every 16 (g = lane / 16), for both operands alike, which only reorders the sum.
// Measured, 2048 x 2048 x 3000 on a 2 x 4 mesh: 522 us with scalar FMA, 315 with loads one step ahead and conditions inside
// the loop (every wait then a full one), 229 now: 110 TFLOP/s; MFMA busy for 81 % of the cycles in which a compute unit has
// work, which is 86 % of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_basic.h"
#include "plan.h"
#include "tile_index.h"

namespace gspmd {

constexpr int kF32Tile = 64, kF32BK = 32, kF32Threads = 256;
constexpr int kF32PitchKC = kF32BK + 4;       // K-contiguous operand in LDS: [64][32 k], rows 16 bytes apart in banks
constexpr int kF32PitchKM = kF32Tile + 4;     // K-major operand: [32 k][64], rows 4 k apart 16 banks apart
constexpr int kF32PartFloats = kF32Tile * kF32PitchKC;         // the larger of the two formats (2304; K-major 2176)

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// LEAN: registers for four workgroups on a compute unit.
template <int LAYOUT, bool LEAN>
__global__ __launch_bounds__(kF32Threads, LEAN ? 4 : 1) void dot_f32_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
  __shared__ __attribute__((aligned(16))) float lds[2][2][kF32PartFloats];      // [buffer][operand]
  typedef GSPMD_GLOBAL const float* gfloats;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
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

  // this thread's two 16-byte chunks of an operand's [64][32 k] or [32 k][64] part of a K step: index along m or n, along k
  auto place = [&](bool kmajor, int j, int& x, int& k) {
    const int c = j * kF32Threads + t;
    if (kmajor) { k = c >> 4; x = (c & 15) * 4; } else { x = c >> 3; k = (c & 7) * 4; }
  };
  auto put = [&](bool kmajor, float* part, const f32x4 (&r)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int x, k;
      place(kmajor, j, x, k);
      *reinterpret_cast<f32x4*>(part + (kmajor ? k * kF32PitchKM + x : x * kF32PitchKC + k)) = r[j];
    }
  };
  // four k of the 16-wide fragment that starts at row / column x and k = kb
  auto frag = [&](bool kmajor, const float* part, int x, int kb) -> f32x4 {
    const int xr = x + (lane & 15), kr = kb + (lane >> 4) * 4;
    if (!kmajor) return *reinterpret_cast<const f32x4*>(part + xr * kF32PitchKC + kr);
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = part[(kr + i) * kF32PitchKM + xr];
    return v;
  };

  const gfloats A = (gfloats)P.A, B = (gfloats)P.B;
  // Where a chunk's index along m / n lies beyond the valid extent the last valid row (K-contiguous) or the last four
  // columns (K-major) are loaded in its place: those results are not stored.  A K-major chunk that straddles the end is
  // fetched from the last four columns as well and moved down by `shift` elements.
  gfloats a_at[2], b_at[2];
  int a_shift[2], b_shift[2];
  auto start = [&](bool kmajor, gfloats base, int64_t ld, int x0, int valid, gfloats (&at)[2], int (&shift)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int x, k;
      place(kmajor, j, x, k);
      x += x0;
      const int xs = max(0, min(x, kmajor ? valid - 4 : valid - 1));
      shift[j] = kmajor && x < valid ? x - xs : 0;
      at[j] = base + (kmajor ? k * ld + xs : xs * ld + k);
    }
  };
  start(AKM, A, P.lda, m0, P.Mv, a_at, a_shift);
  start(!BKC, B, P.ldb, n0, P.Nv, b_at, b_shift);
  const bool a_moves = AKM && (P.Mv & 3) && m0 + kF32Tile > P.Mv, b_moves = !BKC && (P.Nv & 3) && n0 + kF32Tile > P.Nv;
  const bool tiny = (AKM && P.Mv < 4) || (!BKC && P.Nv < 4);          // no whole chunk along m or n
  const int64_t a_step = AKM ? static_cast<int64_t>(P.lda) * kF32BK : kF32BK, b_step = BKC ? kF32BK : static_cast<int64_t>(P.ldb) * kF32BK;
  auto load = [&](f32x4 (&ra)[2], f32x4 (&rb)[2]) {                   // the next whole step
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ra[j] = *(GSPMD_GLOBAL const f32x4_any*)a_at[j];
      rb[j] = *(GSPMD_GLOBAL const f32x4_any*)b_at[j];
      a_at[j] += a_step;
      b_at[j] += b_step;
    }
  };
  auto move_down = [](f32x4& v, int s) {
    if (s & 2) v = f32x4{v[2], v[3], 0.f, 0.f};
    if (s & 1) v = f32x4{v[1], v[2], v[3], 0.f};
  };
  // a step that ends beyond the valid K (or an extent below a chunk): element by element, zeros beyond in BOTH operands
  auto load_slow = [&](bool kmajor, gfloats base, int64_t ld, int x0, int valid, int k0, f32x4 (&r)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int x, k;
      place(kmajor, j, x, k);
      x += x0; k += k0;
      r[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int xe = kmajor ? x + e : x, ke = kmajor ? k : k + e;
        if (xe < valid && ke < P.Kv) r[j][e] = base[kmajor ? ke * ld + xe : xe * ld + ke];
      }
    }
  };
  auto publish = [&](int s, const f32x4 (&ra)[2], const f32x4 (&rb)[2]) {
    put(AKM, lds[s][0], ra);
    put(!BKC, lds[s][1], rb);
    __syncthreads();       // (a buffer is written again two steps later, after the barrier of the step between)
  };
  auto multiply = [&](int s) {
    f32x4 fa[2][2], fb[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[h][i] = frag(AKM, lds[s][0], wm + 16 * i, 16 * h);
#pragma unroll
      for (int j = 0; j < 2; ++j) fb[h][j] = frag(!BKC, lds[s][1], wn + 16 * j, 16 * h);
    }
    __builtin_amdgcn_sched_barrier(0);          // all of a step's LDS reads are under way before its first MFMA
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[h][j][q], fa[h][i][q], acc[i][j], 0, 0, 0);
  };
  auto settle = [&](f32x4 (&ra)[2], f32x4 (&rb)[2]) {
    if (a_moves)
#pragma unroll
      for (int j = 0; j < 2; ++j) move_down(ra[j], a_shift[j]);
    if (b_moves)
#pragma unroll
      for (int j = 0; j < 2; ++j) move_down(rb[j], b_shift[j]);
  };

  const int steps = (P.Kv + kF32BK - 1) / kF32BK, whole = tiny ? 0 : P.Kv / kF32BK;
  f32x4 ra[2][2], rb[2][2];                     // loads run two steps ahead
  int s = 0;
  if (whole >= 4) {                             // pairs of steps, their loads without conditions (the waits then count exactly)
    load(ra[0], rb[0]);
    load(ra[1], rb[1]);
    for (; s + 4 <= whole; s += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        settle(ra[h], rb[h]);
        publish(h, ra[h], rb[h]);
        load(ra[h], rb[h]);
        multiply(h);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      settle(ra[h], rb[h]);
      publish(h, ra[h], rb[h]);
      multiply(h);
    }
    s += 2;
  }
  for (; s < steps; ++s) {                      // what is left: at most three whole steps and a partial one
    if (s < whole) {
      load(ra[0], rb[0]);
      settle(ra[0], rb[0]);
    } else {
      load_slow(AKM, A, P.lda, m0, P.Mv, s * kF32BK, ra[0]);
      load_slow(!BKC, B, P.ldb, n0, P.Nv, s * kF32BK, rb[0]);
    }
    publish(s & 1, ra[0], rb[0]);
    multiply(s & 1);
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
