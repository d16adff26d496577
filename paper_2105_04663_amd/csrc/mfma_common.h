// Types and small device helpers shared by the bf16 MFMA kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gspmd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short short4_t;
typedef __attribute__((ext_vector_type(8))) short short8_t;
typedef __attribute__((ext_vector_type(16))) float float16_t;
typedef __attribute__((ext_vector_type(4))) float float4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((address_space(3))) short4_t lds_short4_t;

// s_waitcnt immediate for gfx9: vmcnt [3:0]+[15:14], expcnt [6:4], lgkmcnt [11:8]
constexpr int waitcnt_imm(int vm, int lgkm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 15) << 8); }
constexpr int waitcnt_vm(int vm) { return waitcnt_imm(vm, 15); }      // vmcnt alone
constexpr int waitcnt_lgkm(int lgkm) { return waitcnt_imm(63, lgkm); }  // lgkmcnt alone
#define GSPMD_WAIT_ALL() __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0))

// 16 bytes per lane from sbase + voff (bytes) straight into LDS at lds_addr + lane*16.  The compiler
// does not see this as an LDS write: every consumer is ordered by an explicit s_waitcnt vmcnt + barrier.
__device__ __forceinline__ void global_to_lds16(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}

// the same from an address of every lane's own
__device__ __forceinline__ void global_to_lds16(uint64_t from, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds_addr), "v"(from) : "memory", "m0");
}

// This lane's number in its wave, worked out where it is asked for: what derives from it is neither kept in registers from earlier on nor moved out of a loop.
__device__ __forceinline__ int lane_now() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

// Between staging in a wave's slice of LDS and reading there what other lanes have staged, and before the next staging.  A wave's LDS accesses are carried out
// in the order of the code, so nothing waits; but the compiler sees one lane, for which a store and a read at other addresses may change places.
__device__ __forceinline__ void staged_in_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ u32x4_t mask_tail8(u32x4_t v, int keep) {   // keep first `keep` of 8 bf16
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t m = (2 * d + 1 < keep) ? 0xffffffffu : ((2 * d < keep) ? 0x0000ffffu : 0u);
    v[d] &= m;
  }
  return v;
}

// 16 bytes at an address that is a multiple of 4
typedef uint32_t u32x4_words_t __attribute__((ext_vector_type(4), aligned(4)));

typedef uint32_t u32x4_elements_t __attribute__((ext_vector_type(4), aligned(2)));      // at any bf16 element's address

// Rows of whole 32-bit words that are not padded to 16 bytes: a 16-byte chunk may reach past a row's end.
__host__ __device__ __forceinline__ bool loose_rows(const void* p, int ld) { return (reinterpret_cast<uintptr_t>(p) & 15) || (ld & 7); }

// Eight consecutive k of a K-contiguous row, of which `valid` (any number) exist: zeros beyond, and no word read that holds no valid element.
__device__ __forceinline__ u32x4_t load_k_chunk(__attribute__((address_space(1))) const uint32_t* at, int valid) {
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (valid >= 8) {
    v = *(__attribute__((address_space(1))) const u32x4_words_t*)at;
  } else if (valid > 0) {
#pragma unroll
    for (int d = 0; d < 4; ++d)
      if (2 * d < valid) v[d] = at[d];
    v = mask_tail8(v, valid);
  }
  return v;
}

// the same in rows at any element's address
__device__ __forceinline__ u32x4_t load_k_elements(__attribute__((address_space(1))) const uint16_t* at, int valid) {
  u32x4_t v = {0u, 0u, 0u, 0u};
  if (valid >= 8) {
    v = *(__attribute__((address_space(1))) const u32x4_elements_t*)at;
  } else {
#pragma unroll
    for (int e = 0; e < 7; ++e)
      if (e < valid) v[e >> 1] |= static_cast<uint32_t>(at[e]) << ((e & 1) * 16);
  }
  return v;
}

}  // namespace gspmd
