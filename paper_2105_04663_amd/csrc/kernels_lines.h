// The end of a bf16 MFMA kernel: a wave's 16 x 16 accumulator blocks, 64 columns wide, out to global memory in whole lines.  In the accumulators'
// own order (a lane holds columns n .. n + 3 of row m of a block) an instruction stores 32 bytes (bf16) or 64 (float32) of each of 16 rows;
// staged through the wave's own slice of LDS it stores 16 bytes per lane, lines of 128 or 256 bytes, at the output's element alignment.
// dot_mid_kernel's tiles all end at about the same time, so what their stores take is time that nothing hides.  Measured there (us, in the accumulators' order / whole lines, both
// revisions in turn on one card): 2048 x 1024 x 2048 12.4 / 10.6, 1500 x 512 x 3000 13.5 / 11.8, four of 1000 x 768 x 1024 12.2 / 9.5, six of 601 x 1203 x 697 20.0 / 17.8, sums of
// 2048 x 8192 x 2048 over 4 members 63.3 / 61.1 and over 2, two groups, 62.4 / 60.3; float32 outputs 2048 x 1024 x 4096 20.9 / 20.0.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kernels_basic.h"
#include "mfma_common.h"
#include "plan.h"

namespace gspmd {

template <typename TOut> constexpr int line_pitch() { return 64 * static_cast<int>(sizeof(TOut)) + 16; }
// LDS bytes of a wave that stages `blocks` rows of blocks at once
template <typename TOut> constexpr int line_slice(int blocks) { return blocks * 16 * line_pitch<TOut>(); }

// How whole tiles are stored (others, and rows that may start at odd addresses, as kLinesPlain).
// kLinesThrough, dot_mid_kernel's bf16 outputs: written through to the memory side, where the next kernel finds them.  Left in the caches of the XCDs (kLinesPlain) they are
// written back when the launch ends, which takes 0.4 to 0.7 us; past all caches (kLinesPast) the next kernel fetches them from HBM.  A product and one that reads it (us, plain / past /
// through): 1024 x 2048 x 4096, then x 2048 48.2 / 55.1 / 47.4, 2048 x 1024 x 2048, then x 1024 31.2 / 33.4 / 30.6; sums over members 2048 x 8192 x 2048 over 4, then x 1024 83.2 / 85.7 /
// 82.0, 4096 x 4096 x 2048 over 2, then x 512 78.3 / 82.7 / 77.3; the first product alone 20.9 / 20.2 / 19.9, the first sum 66.8 / 66.0 / 66.0.
// Of a launch that asks for it (`past`) they go past all caches as well: outputs of more than kPastBytes, which the caches do not hold (us, through / past: 64 MB
// in 8 of 2048 x 300 x 2048 31.1 / 31.5; 128 MB in 8 of 4096 x 200 x 2048 67.9 / 51.2, 16384 x 256 x 4096 57.5 / 48.1; 256 MB in 32 of 2048 x 128 x 2048 102.8 / 77.0).
// Rows that are not whole lines of 128 bytes apart are left in the caches all the same, which put together the parts of a line that two stores, often of two workgroups, write (us,
// through / plain, then with a product of x 512 that reads them): 3940 x 1536 x 1984 on 2 x 4 29.0 / 28.3, 52.0 / 51.4; 5079 x 100 x 934 on 2 x 3, dense, 8.9 / 8.3, 24.8 / 24.1; 4925 x 552 x 928 16.1 /
// 15.9, 36.8 / 36.6; 3994 x 1216 x 1063 on 2 x 4 21.1 / 20.8, 39.7 / 39.0.
// kLinesPast, dot_pair_kernel's bf16 outputs, launches of many tiles: four experts' weight gradients of 4096 x 8192, K 384 109 us, plain 140, and with an update that reads them 262, 281; of
// 2048 x 4096, K 2048 29.8, 31.0 and 39.1, 39.5.
// kLinesPlain where rows start at odd addresses and lines are stored in two parts (601 x 1203 x 697 17.9, past 18.4), and float32 outputs, mostly partial sums that the next kernel
// reads (4096 x 512 x 2048, four times with their sum, 79.2, past 81.2).
enum LineStores { kLinesPlain, kLinesPast, kLinesThrough };

// Block (i, j) of BLOCKS x 4 is value(i, j); the wave's first row and column are row0 and col0.  `inside`: all of the workgroup's tile is valid.
template <typename TOut, int BLOCKS, int AT_ONCE, LineStores STORES, typename Value>
__device__ __forceinline__ void store_lines(unsigned char* slice, GSPMD_GLOBAL TOut* C, const Problem& P, int row0, int col0, bool inside, int epilogue, int lane, Value value, bool past = false) {
  constexpr int V = 16 / static_cast<int>(sizeof(TOut)), kLanes = 64 / V, kRowsAt = 64 / kLanes;       // columns of a lane, lanes of a row, rows of a store
  constexpr int kPitch = line_pitch<TOut>();
  typedef TOut out_vec __attribute__((ext_vector_type(V), aligned(sizeof(TOut))));
  typedef unsigned int line_t __attribute__((vector_size(16)));
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
#pragma unroll
  for (int pass = 0; pass < BLOCKS / AT_ONCE; ++pass) {
    auto stage = [&](auto relu_tag) {           // (Relu or not is decided once: inside the loop it becomes a compare and a select per element)
      constexpr int32_t kEpilogue = decltype(relu_tag)::value ? GSPMD_EPILOGUE_RELU : GSPMD_EPILOGUE_NONE;
#pragma unroll
      for (int b = 0; b < AT_ONCE; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4_t x = value(pass * AT_ONCE + b, j);
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = apply_epilogue(x[e], kEpilogue);
          unsigned char* at = slice + (b * 16 + (lane & 15)) * kPitch + (j * 16 + (lane >> 4) * 4) * sizeof(TOut);
          if constexpr (sizeof(TOut) == 2)
            *reinterpret_cast<bf16x4_t*>(at) = bf16x4_t{static_cast<__bf16>(v[0]), static_cast<__bf16>(v[1]), static_cast<__bf16>(v[2]), static_cast<__bf16>(v[3])};
          else
            *reinterpret_cast<float4_t*>(at) = float4_t{v[0], v[1], v[2], v[3]};
        }
    };
    if (epilogue == GSPMD_EPILOGUE_RELU) stage(std::true_type{}); else stage(std::false_type{});
    staged_in_order();
    const int row = row0 + pass * AT_ONCE * 16 + lane / kLanes, col = col0 + lane % kLanes * V;
    GSPMD_GLOBAL TOut* const c0 = C + static_cast<int64_t>(row) * P.ldc + col;
    const int keep = min(V, P.Nv - col), room = min(V, P.Ns - col);
    constexpr int kStores = AT_ONCE * 16 / kRowsAt;
    auto staged = [&](int p) { return *reinterpret_cast<const u32x4_t*>(slice + (p * kRowsAt + lane / kLanes) * kPitch + lane % kLanes * 16); };
    auto store = [&](GSPMD_GLOBAL TOut* c, u32x4_t v) {
      if constexpr (STORES == kLinesPast) __builtin_nontemporal_store(__builtin_bit_cast(out_vec, v), (GSPMD_GLOBAL out_vec*)c);
      else if constexpr (STORES == kLinesThrough) __builtin_amdgcn_global_store_b128((GSPMD_GLOBAL line_t*)c, __builtin_bit_cast(line_t, v), "agent");
      else *(GSPMD_GLOBAL out_vec*)c = __builtin_bit_cast(out_vec, v);
    };
    // One read, one store (with all reads first four experts' weight gradients of 4096 x 8192 took 116.6 us, so 114.9); outputs written through all reads first (backward of
    // 2048 x 2048 x 8192 on 2 x 2 146.2 us, so 144.1).
    constexpr bool kReadsFirst = STORES == kLinesThrough;
    const bool rows_are_lines = !(((static_cast<uint32_t>(P.ldc) * static_cast<uint32_t>(sizeof(TOut))) | static_cast<uint32_t>(reinterpret_cast<uintptr_t>(P.C))) & 127);
    if (kReadsFirst && inside) {
      u32x4_t v[kStores];
#pragma unroll
      for (int p = 0; p < kStores; ++p) v[p] = staged(p);
      if (past)
#pragma unroll
        for (int p = 0; p < kStores; ++p) {
          asm volatile("" ::: "memory");        // (or the compiler makes one store of the three, without the hint)
          __builtin_nontemporal_store(__builtin_bit_cast(out_vec, v[p]), (GSPMD_GLOBAL out_vec*)(c0 + static_cast<int64_t>(p) * kRowsAt * P.ldc));
          asm volatile("" ::: "memory");
        }
      else if (!rows_are_lines)
#pragma unroll
        for (int p = 0; p < kStores; ++p) {
          asm volatile("" ::: "memory");
          *(GSPMD_GLOBAL out_vec*)(c0 + static_cast<int64_t>(p) * kRowsAt * P.ldc) = __builtin_bit_cast(out_vec, v[p]);
          asm volatile("" ::: "memory");
        }
      else
#pragma unroll
        for (int p = 0; p < kStores; ++p) store(c0 + static_cast<int64_t>(p) * kRowsAt * P.ldc, v[p]);
    } else {
#pragma unroll
      for (int p = 0; p < kStores; ++p) {
        u32x4_t v = staged(p);
        GSPMD_GLOBAL TOut* const c = c0 + static_cast<int64_t>(p) * kRowsAt * P.ldc;
        if (!kReadsFirst && inside) {
          store(c, v);
          continue;
        }
        if (row + p * kRowsAt >= P.Mv || room <= 0) continue;
        if constexpr (sizeof(TOut) == 2) {
          v = mask_tail8(v, keep);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (e >= keep) v[e] = 0u;
        }
        const out_vec o = __builtin_bit_cast(out_vec, v);
        if (room == V) *(GSPMD_GLOBAL out_vec*)c = o;
        else
#pragma unroll
          for (int e = 0; e < V; ++e) if (e < room) c[e] = o[e];
      }
    }
    staged_in_order();                          // the next pass stages into what this one reads
  }
}

}  // namespace gspmd
