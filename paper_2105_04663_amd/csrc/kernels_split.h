// bf16 MFMA contraction for products too small to give every compute unit a 256 x 256 tile: few rows (decoding), few
// output tiles, or operands of any alignment.  C[m,n] = sum_k A[m,k] * B[k,n] like dot_mfma_kernel, in tiles of 16 RB
// rows x 16 CB columns whose K range is split over the eight waves of a workgroup.
//
// What bounds it: with few rows the rhs (weights) streams from HBM once and little is computed per byte, so the kernel
// has to keep enough bytes in flight on enough compute units; with few output tiles it is the length of one wave's chain
// of K steps.  Both call for small tiles and for splitting K inside the workgroup, where the partial sums meet in LDS and
// no workspace, counter or second launch is needed.  Wave w takes the 32-wide K steps w, w + 8, w + 16, ..: it loads its
// own operand pieces into registers, DEPTH steps ahead, passes them through its own piece of LDS into fragment layout (a
// K-major operand with the transpose read), and shares nothing with the other waves until the end, so the loop has no
// barrier.  The eight waves' accumulators are added in wave order, in fp32.
//
// Loads are 16 bytes at any element alignment.  An operand chunk never reaches past a row's valid end unless rows are
// padded to 8 elements: the last tile of an unpadded K-major operand is moved back so that it ends at the last valid
// column (the columns that it shares with its neighbour are computed twice, in the same order); of one narrower than a tile the
// last chunk is fetched early and moved down in registers (element by element: 32 of 268 x 2185 x 11 73 us, now 24; of 56 x 1562 x 13 33, now 13).  What is left of K
// after the 32-wide steps, or an extent of fewer than 8, goes element by element.
//
// Measured (us, weights not in cache; before: 256 x 256 tiles on 32 to 128 of the 256 compute units): 32 x 8192 x 8192
// 101 -> 43 (134 MB of weights at 3.1 TB/s; 36 with rows of 8256 elements, a power of two costs the L2 channels), 64 rows
// 105 -> 47, 256 rows 135 -> 97, 16 x 8192 x 32768 -> 115 (4.7 TB/s), 256 x 2048 x 2048 39 -> 13, 64 x 1024 x 1024 14 -> 6.
// Of the 43 us, 40 are the loads alone (36 with the tiles' order below: 32 x 8192 x 8192 42.7 -> 40.1, 16 rows 44.0 -> 42.8, 128 x 4096 x
// 4096 16.5 -> 15.1).  Running further ahead (9 instead of 6 steps, or only 2) changes nothing: a compute unit's L1 keeps about 105 lines of 128 bytes
// in flight, 608 cycles each at 32 x 8192 x 8192 (256 workgroups: two row tiles draw every weight panel, 268 MB from L2, 144
// from HBM), and stalls on them for half of its cycles; the matrix cores are busy for 7 %, LDS for 25 %.
// Tiles of 32 columns read half lines, but are twice as many: where 64 columns leave compute units without a tile they are a fifth to a quarter
// faster (16 x 3648 x 2081 13.9 -> 11.4, 18 x 2944 x 1306 10.6 -> 8.2, 8 x 4096 x 1024 10.3 -> 7.6, 16 x 8192 x 8192 41.7 -> 38.4, 172 x 2361 x 559 14.7 -> 10.9).  16 columns
// gain another 4 to 9 % with few dozen tiles only, sixteen waves nothing.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "kernels_basic.h"
#include "launch.h"
#include "plan.h"
#include "tile_index.h"

namespace gspmd {

typedef __attribute__((ext_vector_type(8))) __bf16 split_bf16x8;
typedef __attribute__((ext_vector_type(4))) short split_short4;
typedef __attribute__((ext_vector_type(8))) short split_short8;
typedef __attribute__((address_space(3))) split_short4 lds_split_short4;
typedef __attribute__((ext_vector_type(4))) float split_f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t split_u32x4;
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));     // 16 bytes at a bf16 element's alignment

// How far ahead (in K steps of a wave) operands are loaded: as deep as the 256 registers of a wave allow.
template <int RB, int CB> constexpr int split_depth() { return RB == 4 ? 4 : RB == 2 ? 5 : 6; }

// LDS bytes of a wave's transposition piece and of the whole workgroup
template <int RB, int CB> constexpr int split_piece() { return (RB + CB) * 1024; }
constexpr int kSplitQuad = 4 * 272;            // one 16 x 16 block of fp32 in the reduction: four 16-lane groups of 256 bytes, 16 apart
template <int RB, int CB> constexpr int split_lds() {
  constexpr int pieces = kSplitWaves * split_piece<RB, CB>(), sums = kSplitWaves * RB * CB * kSplitQuad;
  return pieces > sums ? pieces : sums;
}

// Transposition piece of a K-major operand: [32 k][16 W columns], 2 W chunks of 16 bytes per k row.  Chunk pairs (the 16
// columns of one block) are XOR-swizzled by the row so that the 4 rows x 32 bytes that a 16-lane group reads, and those of
// the group beside it (8 rows further), lie in different banks.
template <int W> __device__ __forceinline__ int split_pair(int block, int krow) {
  if constexpr (W >= 4) return block ^ (((krow >> 1) & 1) | (((krow >> 3) & 1) << 1));
  else if constexpr (W == 2) return block ^ ((krow >> 1) & 1);
  else return block;
}

template <typename TOut, int LAYOUT, int RB, int CB>
__global__ __launch_bounds__(kSplitThreads) void dot_split_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int epilogue, int spread,
                                                                  unsigned long long* __restrict__ timeline, int timeline_records) {
  constexpr bool AKM = (LAYOUT & GSPMD_LAYOUT_LHS_K_MAJOR) != 0, BKC = (LAYOUT & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) != 0;
  constexpr int BM = 16 * RB, BN = 16 * CB, D = split_depth<RB, CB>();
  typedef GSPMD_GLOBAL const unsigned char* gbytes;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  unsigned long long* const rec = timeline_record(timeline, timeline_records);
  if (rec != nullptr) timeline_stamp(rec, 0, t, timeline_where());
  const int tile = spread ? spread_tile(blockIdx.x, gridDim.x) : logical_tile(blockIdx.x, gridDim.x);
  const Problem P = lookup_problem(tab, n_prob, tile);
  const int local = tile - P.tile_begin;
  // the row index runs fastest: the row tiles that share a weight panel are on one XCD at the same time
  const int tiles_m = (P.Mv + BM - 1) / BM;
  const int tile_row = local % tiles_m, tile_col = local / tiles_m;
  const int m_nom = tile_row * BM, n_nom = tile_col * BN;             // where the tile's share of the output begins
  // rows padded to 8 elements may be read up to there
  const bool a_pad = !((reinterpret_cast<uintptr_t>(P.A) & 15) | (P.lda & 7)), b_pad = !((reinterpret_cast<uintptr_t>(P.B) & 15) | (P.ldb & 7));
  int m0 = m_nom, n0 = n_nom;
  // an extent too short for whole chunks, or one that ends inside a chunk (in tiles of 32 columns only: 64 x 64 have no registers for it, and the
  // others would be 1 to 3 % slower for every operand)
  constexpr bool kMoves = CB == 2;
  bool slow = false, a_moves = false, b_moves = false;
  if (AKM && !a_pad && m0 + BM > P.Mv) { m0 = max(0, P.Mv - BM); slow = P.Mv < (kMoves ? 8 : BM); a_moves = P.Mv < BM && (P.Mv & 7); }
  if (!BKC && !b_pad && n0 + BN > P.Nv) { n0 = max(0, P.Nv - BN); slow = slow || P.Nv < (kMoves ? 8 : BN); b_moves = P.Nv < BN && (P.Nv & 7); }

  split_f32x4 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = split_f32x4{0.f, 0.f, 0.f, 0.f};

  unsigned char* const piece_a = smem + wave * split_piece<RB, CB>();
  unsigned char* const piece_b = piece_a + RB * 1024;

  // ---- where this lane's chunks are, in bytes from the first element of the tile at k = 0
  uint32_t a_off[RB], b_off[CB];
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    if constexpr (AKM) {
      const int idx = j * 64 + lane, kr = idx / (2 * RB);
      int m = m0 + (idx - kr * (2 * RB)) * 8;
      if (m >= P.Mv) m = ((P.Mv - 1) >> 3) << 3;                      // only where rows are padded, or few: the last chunk again
      if (kMoves && !a_pad) m = min(m, max(0, P.Mv - 8));             // fetched early
      a_off[j] = (static_cast<uint32_t>(kr) * P.lda + m) * 2;
    } else {
      a_off[j] = static_cast<uint32_t>(min(j * 16 + (lane >> 2), P.Mv - 1 - m0)) * static_cast<uint32_t>(P.lda) * 2 + (lane & 3) * 16;
    }
  }
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    if constexpr (!BKC) {
      const int idx = j * 64 + lane, kr = idx / (2 * CB);
      int n = n0 + (idx - kr * (2 * CB)) * 8;
      if (n >= P.Nv) n = ((P.Nv - 1) >> 3) << 3;
      if (kMoves && !b_pad) n = min(n, max(0, P.Nv - 8));
      b_off[j] = (static_cast<uint32_t>(kr) * P.ldb + n) * 2;
    } else {
      b_off[j] = static_cast<uint32_t>(min(j * 16 + (lane >> 2), P.Nv - 1 - n0)) * static_cast<uint32_t>(P.ldb) * 2 + (lane & 3) * 16;
    }
  }
  const gbytes a_base = (gbytes)P.A + (AKM ? int64_t(0) : static_cast<int64_t>(m0) * P.lda * 2);
  const gbytes b_base = (gbytes)P.B + (BKC ? static_cast<int64_t>(n0) * P.ldb * 2 : int64_t(0));
  const int64_t a_step = AKM ? static_cast<int64_t>(P.lda) * 64 : 64, b_step = BKC ? 64 : static_cast<int64_t>(P.ldb) * 64;   // bytes per 32 k

  // This wave's next step: both bases are scalar registers that move on by eight steps.  (Written as base + step * size
  // the compiler keeps a 64-bit address per chunk and lane and adds to every one of them at every step.)
  uint64_t a_at = reinterpret_cast<uint64_t>(a_base) + wave * a_step, b_at = reinterpret_cast<uint64_t>(b_base) + wave * b_step;
  auto load_step = [&](split_u32x4 (&ra)[RB], split_u32x4 (&rb)[CB]) {
    asm volatile("" : "+s"(a_at), "+s"(b_at));
    // (likewise the offsets: their widening to 64 bits must not move out of the loop)
#pragma unroll
    for (int j = 0; j < CB; ++j) asm volatile("" : "+v"(b_off[j]));
#pragma unroll
    for (int j = 0; j < RB; ++j) asm volatile("" : "+v"(a_off[j]));
#pragma unroll
    for (int j = 0; j < CB; ++j) rb[j] = *(GSPMD_GLOBAL const u32x4_any*)((gbytes)b_at + b_off[j]);
#pragma unroll
    for (int j = 0; j < RB; ++j) ra[j] = *(GSPMD_GLOBAL const u32x4_any*)((gbytes)a_at + a_off[j]);
    a_at += kSplitWaves * a_step;
    b_at += kSplitWaves * b_step;
  };
  // the same chunks element by element, zero beyond the valid extents: BOTH operands beyond the valid K
  auto load_step_slow = [&](int step, split_u32x4 (&ra)[RB], split_u32x4 (&rb)[CB]) {
    auto chunk = [&](const void* base, int64_t ld, bool kmajor, int width, int x0, int x_valid, int j) -> split_u32x4 {
      split_u32x4 v = {0u, 0u, 0u, 0u};
      int x, k;                                                       // first element: index along m or n, and along K
      if (kmajor) {
        const int idx = j * 64 + lane, kr = idx / (2 * width);
        x = x0 + (idx - kr * (2 * width)) * 8;
        k = step * 32 + kr;
      } else {
        x = x0 + j * 16 + (lane >> 2);
        k = step * 32 + (lane & 3) * 8;
      }
      GSPMD_GLOBAL const bf16_bits* at = (GSPMD_GLOBAL const bf16_bits*)base;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int xe = kmajor ? x + e : x, ke = kmajor ? k : k + e;
        if (xe < x_valid && ke < P.Kv) {
          const uint32_t bits = at[kmajor ? ke * ld + xe : xe * ld + ke];
          v[e >> 1] |= bits << ((e & 1) * 16);
        }
      }
      asm volatile("" ::: "memory");                                  // one chunk after the other: registers are for the fast path
      return v;
    };
#pragma unroll
    for (int j = 0; j < CB; ++j) rb[j] = chunk(P.B, P.ldb, !BKC, CB, n0, P.Nv, j);
#pragma unroll
    for (int j = 0; j < RB; ++j) ra[j] = chunk(P.A, P.lda, AKM, RB, m0, P.Mv, j);
  };

  // K-major operand: this wave's chunks into its piece, then every block's fragment back, transposed.  The wave's LDS
  // operations execute in order, so no wait is needed between them; the compiler is kept from reordering them.
  auto transpose = [&](auto width_tag, unsigned char* piece, const auto& regs, auto& frags) {
    constexpr int W = decltype(width_tag)::value;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int idx = j * 64 + lane, kr = idx / (2 * W), c = idx - kr * (2 * W);
      *reinterpret_cast<split_u32x4*>(piece + kr * (32 * W) + split_pair<W>(c >> 1, kr) * 32 + (c & 1) * 16) = regs[j];
    }
    asm volatile("" ::: "memory");
    const int kr = (lane >> 4) * 8 + ((lane & 15) >> 2);
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const unsigned char* p = piece + kr * (32 * W) + split_pair<W>(j, kr) * 32 + (lane & 3) * 8;
      split_short8 both;
      both.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_split_short4*)p);
      both.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_split_short4*)(p + 4 * 32 * W));
      frags[j] = __builtin_bit_cast(split_bf16x8, both);
    }
    asm volatile("" ::: "memory");
  };
  // K-contiguous operand: four consecutive lanes bring 64 bytes of a row (a load in fragment layout, a row per lane, takes
  // the address unit four times as long: 16.1 instead of 13.2 us at 256 x 2048 x 2048, both operands K-contiguous);
  // its chunks change lanes in LDS.
  auto relane = [&](auto width_tag, unsigned char* piece, const auto& regs, auto& frags) {
    constexpr int W = decltype(width_tag)::value;
    const int wr = lane >> 2, rr = lane & 15;
#pragma unroll
    for (int j = 0; j < W; ++j) *reinterpret_cast<split_u32x4*>(piece + j * 1024 + wr * 64 + (((lane & 3) ^ swz_a(wr)) << 4)) = regs[j];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < W; ++j)
      frags[j] = __builtin_bit_cast(split_bf16x8, *reinterpret_cast<const split_u32x4*>(piece + j * 1024 + rr * 64 + (((lane >> 4) ^ swz_a(rr)) << 4)));
    asm volatile("" ::: "memory");
  };
  // Chunks of a K-major operand narrower than the tile, the last of them fetched early because it would have reached past the valid extent:
  // moved down to where its elements belong.
  auto move_down = [&](auto width_tag, auto& regs, int valid) {
    constexpr int W = decltype(width_tag)::value;
    int l = lane;
    asm volatile("" : "+v"(l));                                         // (worked out here, not kept in registers through the loop)
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int x = ((j * 64 + l) & (2 * W - 1)) * 8, by = x < valid ? max(0, x + 8 - valid) : 0;
      split_u32x4 v = regs[j];
      if (by & 4) v = split_u32x4{v[2], v[3], 0u, 0u};
      if (by & 2) v = split_u32x4{v[1], v[2], v[3], 0u};
      if (by & 1) v = split_u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
      regs[j] = v;
    }
  };
  auto compute = [&](split_u32x4 (&ra)[RB], split_u32x4 (&rb)[CB], bool whole_step) {
    split_bf16x8 fa[RB], fb[CB];
    if (kMoves && AKM && a_moves && whole_step) move_down(std::integral_constant<int, RB>{}, ra, P.Mv);
    if (kMoves && !BKC && b_moves && whole_step) move_down(std::integral_constant<int, CB>{}, rb, P.Nv);
    if constexpr (BKC) relane(std::integral_constant<int, CB>{}, piece_b, rb, fb);
    else transpose(std::integral_constant<int, CB>{}, piece_b, rb, fb);
    if constexpr (AKM) transpose(std::integral_constant<int, RB>{}, piece_a, ra, fa);
    else relane(std::integral_constant<int, RB>{}, piece_a, ra, fa);
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };

  const int steps = (P.Kv + 31) >> 5, whole = slow ? 0 : P.Kv >> 5;    // K steps, and those of them without predicates
  {
    const int mine = whole > wave ? (whole - wave + kSplitWaves - 1) / kSplitWaves : 0;
    split_u32x4 ra[D][RB], rb[D][CB];
    timeline_stamp(rec, 1, t);
    timeline_stamp(rec, 2, t);
    timeline_stamp(rec, 3, t);
    int i = 0;
    // as long as whole rounds of D steps remain, without conditions: the waits then count exactly and D - 1 steps stay in
    // flight (a conditional load anywhere before makes the compiler wait for everything once a round)
    if (mine >= 2 * D) {
#pragma unroll
      for (int d = 0; d < D; ++d) load_step(ra[d], rb[d]);
      __builtin_amdgcn_sched_barrier(0);
      for (; i + 2 * D <= mine; i += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          compute(ra[d], rb[d], true);
          load_step(ra[d], rb[d]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (d < mine) load_step(ra[d], rb[d]);
    }
    for (; i < mine; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (i + d < mine) compute(ra[d], rb[d], true);
        if (i + d + D < mine) load_step(ra[d], rb[d]);
      }
    }
    for (int s = whole + ((wave - whole) & (kSplitWaves - 1)); s < steps; s += kSplitWaves) {    // the rest of this wave's steps
      load_step_slow(s, ra[0], rb[0]);
      compute(ra[0], rb[0], false);
    }
  }

  // ---- the waves' sums meet in LDS (their transposition pieces are done with) and are added in wave order
  constexpr int kSlotBytes = RB * CB * kSplitQuad;
  timeline_stamp(rec, 4, t);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
      *reinterpret_cast<split_f32x4*>(smem + wave * kSlotBytes + (i * CB + j) * kSplitQuad + (lane >> 4) * 272 + (lane & 15) * 16) = acc[i][j];
  __syncthreads();

  timeline_stamp(rec, 5, t);
  // ---- epilogue: four consecutive columns of a row per thread, 4 CB threads per row
  GSPMD_GLOBAL TOut* const C = (GSPMD_GLOBAL TOut*)P.C;
  typedef TOut out4 __attribute__((ext_vector_type(4), aligned(sizeof(TOut))));
  for (int idx = t; idx < BM * BN / 4; idx += kSplitThreads) {
    const int row = idx / (4 * CB), c4 = idx - row * (4 * CB);
    const int m = m0 + row, n = n0 + c4 * 4;
    const unsigned char* p = smem + ((row >> 4) * CB + (c4 >> 2)) * kSplitQuad + (c4 & 3) * 272 + (row & 15) * 16;
    split_f32x4 s = *reinterpret_cast<const split_f32x4*>(p);
#pragma unroll
    for (int w = 1; w < kSplitWaves; ++w) s += *reinterpret_cast<const split_f32x4*>(p + w * kSlotBytes);
    if (m >= P.Mv || n >= P.Ns) continue;
    out4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = n + e < P.Nv ? apply_epilogue(s[e], epilogue) : 0.f;
      if constexpr (sizeof(TOut) == 2) o[e] = float_to_bf16(v);
      else o[e] = v;
    }
    GSPMD_GLOBAL TOut* c = C + static_cast<int64_t>(m) * P.ldc + n;
    if (n + 4 <= P.Ns) *(GSPMD_GLOBAL out4*)c = o;
    else
#pragma unroll
      for (int e = 0; e < 4; ++e) if (n + e < P.Ns) c[e] = o[e];
  }
  // zeros of the static block: right of a tile that was moved back, and below the last row tile (what lies further
  // down, and whole tile columns of padding, the fill kernel clears)
  const int col_end = min(n_nom + BN, P.Ns);
  const int m_done = min(m_nom + BM, P.Mv);
  if (n0 < n_nom) zero_block<kSplitThreads, TOut>(C, P.ldc, m_nom, m_done, n0 + BN, col_end, t);
  if (m_done == P.Mv) zero_block<kSplitThreads, TOut>(C, P.ldc, P.Mv, rows_cleared(P.Mv, P.Ms), n_nom, col_end, t);
  if (rec != nullptr) {
    timeline_stamp(rec, 6, t);
    __builtin_amdgcn_s_waitcnt(0);
    timeline_stamp(rec, 7, t);
  }
}

template <typename TOut, int LAYOUT, int RB, int CB>
inline bool launch_dot_split_as(const MfmaLaunch& l, hipStream_t stream) {
  constexpr int lds = split_lds<RB, CB>();
  static std::once_flag once[kMaxDevices];
  static bool ok[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::call_once(once[dev], [dev] {
    ok[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(&dot_split_kernel<TOut, LAYOUT, RB, CB>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds) == hipSuccess;
  });
  if (!ok[dev]) return false;
  hipLaunchKernelGGL((dot_split_kernel<TOut, LAYOUT, RB, CB>), dim3(static_cast<unsigned>(l.tiles)), dim3(kSplitThreads), lds, stream, *l.inl, l.tab,
                     l.n_prob, l.epilogue, l.spread ? 1 : 0, l.timeline, l.timeline_records);
  return hipGetLastError() == hipSuccess;
}

template <int LAYOUT, typename TOut>
bool launch_dot_split_out(const MfmaLaunch& l, int row_blocks, int col_blocks, hipStream_t stream) {
  if (col_blocks == 2) return row_blocks == 1 ? launch_dot_split_as<TOut, LAYOUT, 1, 2>(l, stream) : launch_dot_split_as<TOut, LAYOUT, 2, 2>(l, stream);
  switch (row_blocks) {
    case 1: return launch_dot_split_as<TOut, LAYOUT, 1, 4>(l, stream);
    case 2: return launch_dot_split_as<TOut, LAYOUT, 2, 4>(l, stream);
    default: return launch_dot_split_as<TOut, LAYOUT, 4, 4>(l, stream);
  }
}
template <int LAYOUT>
bool launch_dot_split_layout(const MfmaLaunch& l, int32_t out_dtype, int row_blocks, int col_blocks, hipStream_t stream) {
  return out_dtype == GSPMD_F32 ? launch_dot_split_out<LAYOUT, float>(l, row_blocks, col_blocks, stream)
                                : launch_dot_split_out<LAYOUT, bf16_bits>(l, row_blocks, col_blocks, stream);
}

}  // namespace gspmd
