// Device kernels that are not MFMA-shaped: the any-layout fallback contraction (bf16 operands with rows too long for
// 32-bit offsets inside a tile, or at odd byte addresses), the K-partial sum and the shard <-> global copies.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.h"

namespace gspmd {

typedef uint16_t bf16_bits;

__device__ __forceinline__ float bf16_to_float(bf16_bits b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// round-to-nearest-even; NaN stays NaN (quiet bit forced so the payload cannot round to Inf)
__device__ __forceinline__ bf16_bits float_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<bf16_bits>((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<bf16_bits>(u >> 16);
}

template <typename T> __device__ __forceinline__ float load_as_float(const T* p);
template <> __device__ __forceinline__ float load_as_float<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float load_as_float<bf16_bits>(const bf16_bits* p) { return bf16_to_float(*p); }

template <typename T> __device__ __forceinline__ void store_from_float(T* p, float v);
template <> __device__ __forceinline__ void store_from_float<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void store_from_float<bf16_bits>(bf16_bits* p, float v) { *p = float_to_bf16(v); }

// 16-byte accesses with the non-temporal hint, for data that streams through once (partials being summed, shards
// being regathered): on this part a 4-reads-1-write stream moves 6.1-6.2 TB/s with the hint against 5.2-5.5 without.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x4 load_stream4(const float* p) { return __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p)); }
__device__ __forceinline__ void store_stream4(float* p, f32x4 v) { __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(p)); }
__device__ __forceinline__ void store_stream4(bf16_bits* p, f32x4 v) {
  u32x2 b;
  b.x = static_cast<uint32_t>(float_to_bf16(v.x)) | (static_cast<uint32_t>(float_to_bf16(v.y)) << 16);
  b.y = static_cast<uint32_t>(float_to_bf16(v.z)) | (static_cast<uint32_t>(float_to_bf16(v.w)) << 16);
  __builtin_nontemporal_store(b, reinterpret_cast<u32x2*>(p));
}

// Elementwise epilogue on a finished sum (gspmd_epilogue); NaN stays NaN.
__device__ __forceinline__ float apply_epilogue(float v, int epilogue) {
  return (epilogue == GSPMD_EPILOGUE_RELU && v < 0.f) ? 0.f : v;
}

// Which problem owns output tile `tile`: the last entry whose tile_begin <= tile.
__device__ __forceinline__ int find_problem(const Problem* __restrict__ tab, int n_prob, int tile) {
  int lo = 0, hi = n_prob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab[mid].tile_begin <= tile) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Launch tables small enough to travel as kernel arguments (no upload, so such a launch can be recorded into a HIP
// graph): up to kInlineProblems problems and kInlineRects zero-fill rectangles.  Larger tables are read from device
// memory (`tab` non-null).
constexpr int kInlineProblems = 32;
constexpr int kInlineRects = 2 * kInlineProblems;
struct InlineProblems { Problem p[kInlineProblems]; };
struct InlineRects { ZeroRect r[kInlineRects]; };

// The kernel-argument segment, read in place: loads from it with a wave-uniform index are scalar loads.  (A by-value
// struct parameter that is indexed dynamically through its C++ name is first copied to private memory.)  The table
// read this way must be the kernel's FIRST parameter, which sits at offset 0 of the segment.
#define GSPMD_KERNARG __attribute__((address_space(4)))
#define GSPMD_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const GSPMD_KERNARG T* first_kernel_argument() {
  return (const GSPMD_KERNARG T*)__builtin_amdgcn_kernarg_segment_ptr();
}
template <typename T>
__device__ __forceinline__ T copy_from_kernarg(const GSPMD_KERNARG T* p) {
  static_assert(sizeof(T) % 8 == 0, "copied as 64-bit words");
  const GSPMD_KERNARG uint64_t* q = (const GSPMD_KERNARG uint64_t*)p;
  uint64_t w[sizeof(T) / 8];
#pragma unroll
  for (size_t i = 0; i < sizeof(T) / 8; ++i) w[i] = q[i];
  T out;
  __builtin_memcpy(&out, w, sizeof(T));
  return out;
}

// The problem that owns output tile `tile`: its place in the table in device memory if there is one, else in the table in
// the kernel arguments (an InlineProblems as first parameter), and an entry of whichever table that is.
__device__ __forceinline__ int lookup_problem_index(const Problem* __restrict__ tab, int n_prob, int tile) {
  if (tab) return find_problem(tab, n_prob, tile);
  if (n_prob == 1) return 0;
  // One load and a ballot: a search takes five dependent ones in a table of 32, a microsecond before every tile (4 x 8 mesh of 5998 x 3072 x 9999, 3.75 tiles
  // a compute unit: 286.1 -> 283.8 us on one card; six of 601 x 1203 x 697 20.13 -> 19.84).
  static_assert(kInlineProblems <= 64, "a lane for every problem");
  const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int begin = first_kernel_argument<Problem>()[min(lane, n_prob - 1)].tile_begin;
  return __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n_prob && begin <= tile)) - 1;
}
__device__ __forceinline__ Problem problem_at(const Problem* __restrict__ tab, int i) {
  return tab ? tab[i] : copy_from_kernarg(first_kernel_argument<Problem>() + i);
}
__device__ __forceinline__ Problem lookup_problem(const Problem* __restrict__ tab, int n_prob, int tile) {
  return problem_at(tab, lookup_problem_index(tab, n_prob, tile));
}

// Profiling aid (gspmd_set_tile_timeline): one record of eight 64-bit words per workgroup, written by its thread 0.
// Words 0-7 hold the 100 MHz constant-rate counter at: kernel entry (bits 52-63: XCD id << 8 | compute-unit bits
// 8-15 of the hardware id register), tile decoded, first tile loads issued, first tiles landed (K loop starts), K
// loop left, epilogue starts (leftover K and joined sums done), stores issued, stores complete.  `rec` is null
// when the timeline is off; the branch is uniform and costs two scalar instructions per stamp.
constexpr int kTimelineWords = 8;
__device__ __forceinline__ unsigned long long* timeline_record(unsigned long long* timeline, int records) {
  return (timeline != nullptr && static_cast<int>(blockIdx.x) < records) ? timeline + static_cast<size_t>(blockIdx.x) * kTimelineWords : nullptr;
}
// what word 0 holds beside the time: where the workgroup runs
__device__ __forceinline__ unsigned timeline_where() {
  return ((__builtin_amdgcn_s_getreg((31 << 11) | 20) & 15u) << 8) | ((__builtin_amdgcn_s_getreg((31 << 11) | 4) >> 8) & 255u);
}
__device__ __forceinline__ void timeline_stamp(unsigned long long* rec, int word, int t, unsigned long long tag = 0) {
  if (rec == nullptr) return;
  unsigned long long now;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_memrealtime %0\n\ts_waitcnt lgkmcnt(0)" : "=s"(now) :: "memory");
  if (t == 0) rec[word] = now | (tag << 52);
}

// Zeros over rows [r0, r1) x columns [c0, c1), at most 128 of them, of an output block, by THREADS threads: 16-byte stores at
// element alignment, a power of two of lanes per row.  (Element stores with a division each made the rows below an
// expert's occupied slots cost 25 us of a 27 us launch: 4 experts x 969 slots, 1280 x 1088.)
template <int THREADS, typename TOut>
__device__ __forceinline__ void zero_block(GSPMD_GLOBAL TOut* C, int64_t ldc, int r0, int r1, int c0, int c1, int t) {
  constexpr int V = 16 / static_cast<int>(sizeof(TOut)), kLanes = 128 / V;
  typedef TOut vec __attribute__((ext_vector_type(16 / sizeof(TOut)), aligned(sizeof(TOut))));
  const int c = c0 + (t % kLanes) * V;
  if (c >= c1) return;
  for (int r = r0 + t / kLanes; r < r1; r += THREADS / kLanes) {
    GSPMD_GLOBAL TOut* at = C + r * ldc + c;
    if (c + V <= c1) *(GSPMD_GLOBAL vec*)at = vec(TOut(0));
    else
      for (int e = 0; c + e < c1; ++e) at[e] = TOut(0);
  }
}

constexpr int kGenTile = 64;   // output tile edge of the fallback kernel
constexpr int kGenBK = 16;

// Fallback contraction: 64x64 output tile per workgroup, 4x4 outputs per thread, fp32 FMA.
// Every load is predicated on the valid extents (masked positions contribute 0 and are never
// read); stores cover the static extents and write 0 outside the valid region.
template <typename TIn, typename TOut>
__global__ __launch_bounds__(256) void dot_fallback_kernel(const InlineProblems inl, const Problem* __restrict__ tab, int n_prob, int layout, int epilogue) {
  __shared__ float As[kGenBK][kGenTile + 4];   // [k][m]
  __shared__ float Bs[kGenBK][kGenTile + 4];   // [k][n]
  const int tile = blockIdx.x;
  const Problem P = lookup_problem(tab, n_prob, tile);
  const int local = tile - P.tile_begin;
  const int m0 = (local / P.tiles_n) * kGenTile, n0 = (local % P.tiles_n) * kGenTile;
  const TIn* __restrict__ A = static_cast<const TIn*>(P.A);
  const TIn* __restrict__ B = static_cast<const TIn*>(P.B);
  TOut* __restrict__ C = static_cast<TOut*>(P.C);
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  // element strides of the two indices of each operand
  const int64_t a_sm = (layout & GSPMD_LAYOUT_LHS_K_MAJOR) ? 1 : P.lda, a_sk = (layout & GSPMD_LAYOUT_LHS_K_MAJOR) ? P.lda : 1;
  const int64_t b_sk = (layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) ? 1 : P.ldb, b_sn = (layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) ? P.ldb : 1;
  if (m0 < P.Mv && n0 < P.Nv) {
    const int am = t >> 2, ak = (t & 3) * 4;     // A: row am, 4 consecutive k
    const int bk = t >> 4, bn = (t & 15) * 4;    // B: row bk, 4 consecutive n
    for (int k0 = 0; k0 < P.Kv; k0 += kGenBK) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int m = m0 + am, k = k0 + ak + j;
        As[ak + j][am] = (m < P.Mv && k < P.Kv) ? load_as_float<TIn>(A + m * a_sm + k * a_sk) : 0.f;
        const int kk = k0 + bk, n = n0 + bn + j;
        Bs[bk][bn + j] = (kk < P.Kv && n < P.Nv) ? load_as_float<TIn>(B + kk * b_sk + n * b_sn) : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kGenBK; ++k) {
        float a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { a[i] = As[k][ty * 4 + i]; b[i] = Bs[k][tx * 4 + i]; }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= P.Ms) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= P.Ns) continue;
      const float v = (m < P.Mv && n < P.Nv) ? apply_epilogue(acc[i][j], epilogue) : 0.f;
      store_from_float<TOut>(C + static_cast<int64_t>(m) * P.ldc + n, v);
    }
  }
}

// Zero fill of the parts of static output blocks that lie in whole tiles beyond the valid extents.
// grid.y = rectangle, grid.x strides over its 16-byte vectors (VEC elements; the host picks VEC = 1 unless the
// pointers, leading dimensions, first columns and widths of all rectangles allow 16-byte stores).
template <typename TOut, int VEC>
__global__ __launch_bounds__(256) void zero_rects_kernel(const InlineRects inl, const ZeroRect* __restrict__ rects) {
  const ZeroRect R = rects ? rects[blockIdx.y] : copy_from_kernarg(first_kernel_argument<ZeroRect>() + blockIdx.y);
  const int wv = (R.c1 - R.c0) / VEC;
  const int64_t total = static_cast<int64_t>(R.r1 - R.r0) * wv;
  TOut* __restrict__ C = static_cast<TOut*>(R.C);
  struct alignas(sizeof(TOut) * VEC) Vec { TOut v[VEC]; };
  Vec z;
#pragma unroll
  for (int j = 0; j < VEC; ++j) z.v[j] = TOut(0);
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = i / wv;
    const int c = static_cast<int>(i - r * wv) * VEC;
    *reinterpret_cast<Vec*>(C + (R.r0 + r) * R.ldc + R.c0 + c) = z;
  }
}

// Arrival counters of joined output tiles start every launch at zero (a fill kernel rather than a memset node, so
// that the call can be recorded into a HIP graph).
static __global__ __launch_bounds__(256) void zero_words_kernel(uint32_t* __restrict__ words, int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    words[i] = 0u;
}

// ---------------------------------------------------------------------------------------
// Sum of K-partials (the arithmetic of the AllReduce along a contracting mesh dimension).
// ---------------------------------------------------------------------------------------
constexpr int kMaxPartials = 16;
struct PartialPtrs { const float* p[kMaxPartials]; };

// rows x cols fp32 partials with leading dimension ld_in -> out with leading dimension ld_out.
// VEC = 4: cols, both leading dimensions and all pointers allow 16-byte (fp32) accesses.
template <typename TOut, int VEC>
__global__ __launch_bounds__(256) void reduce_partials_kernel(PartialPtrs ptrs, int n_partials,
                                                              int64_t rows, int64_t cols, int64_t ld_in,
                                                              TOut* __restrict__ out, int64_t ld_out) {
  const int64_t cols_v = cols / VEC;
  const int64_t total = rows * cols_v;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = i / cols_v, c = (i - r * cols_v) * VEC;
    float acc[VEC];
    if constexpr (VEC == 4) {
      f32x4 sum = load_stream4(ptrs.p[0] + r * ld_in + c);
      for (int p = 1; p < n_partials; ++p) sum += load_stream4(ptrs.p[p] + r * ld_in + c);   // fixed ascending order: deterministic
      store_stream4(out + r * ld_out + c, sum);
    } else {
      acc[0] = ptrs.p[0][r * ld_in + c];
      for (int p = 1; p < n_partials; ++p) acc[0] += ptrs.p[p][r * ld_in + c];
      store_from_float<TOut>(out + r * ld_out + c, acc[0]);
    }
  }
}

// Sum of K-partials written to an out shard that may be a slice of the partials' extent (ReduceScatter: the sum
// followed by each partition's DynamicSlice), any rank.  The last dimension is contiguous on both sides.
struct ScatterDesc {
  int32_t rank;
  int32_t rows;                  // product of the out shard's static extents except the last
  int32_t shard[kMaxRank];       // out shard, static extents
  int32_t log_lanes, unused;     // 2^log_lanes lanes walk along a row of the out shard
  int64_t in_stride[kMaxRank];   // element strides of the (dense) partials
  int64_t out_stride[kMaxRank];  // element strides of the out shard
};
struct ScatterOut {              // one per out shard that a launch writes
  void* out;
  int32_t valid[kMaxRank];       // valid extents (the rest is written as 0 and never read from the partials)
  int64_t in_off[kMaxRank];      // where the out shard starts inside the partial, per dimension
};
struct ScatterLaunch {
  ScatterDesc d;
  PartialPtrs ptrs;
  ScatterOut o[kMaxPartials];
};
static_assert(sizeof(ScatterLaunch) + 2 * sizeof(int) <= 4096 && sizeof(ScatterOut) % 8 == 0, "kernel arguments");

// 2^log_lanes lanes side by side in a row, grid.x covering it in vectors of VEC, the workgroup's other lanes in the next rows; grid.y strides over
// the rows, grid.z = out shard (the slices of one sum in one launch: eight kernels of 2.5 us each before).  Four partials are loaded before
// they are added.  VEC = 4 needs 16-byte aligned pointers and every stride, offset and extent of the last two dimensions a multiple of 4.
template <typename TOut, int VEC>
__global__ __launch_bounds__(256) void reduce_scatter_kernel(const ScatterLaunch launch, int n_partials, int epilogue) {
  const GSPMD_KERNARG ScatterLaunch* const args = first_kernel_argument<ScatterLaunch>();
  const GSPMD_KERNARG ScatterDesc& d = args->d;
  const GSPMD_KERNARG ScatterOut& shard = args->o[blockIdx.z];
  typedef float vec_t __attribute__((ext_vector_type(VEC)));
  GSPMD_GLOBAL TOut* const out = (GSPMD_GLOBAL TOut*)shard.out;
  const int last = d.rank - 1, lane = threadIdx.x & ((1 << d.log_lanes) - 1), rows_side = 256 >> d.log_lanes;
  const int c = ((blockIdx.x << d.log_lanes) + lane) * VEC;
  if (c >= d.shard[last]) return;
  for (int64_t at = static_cast<int64_t>(blockIdx.y) * rows_side + (threadIdx.x >> d.log_lanes); at < d.rows; at += static_cast<int64_t>(gridDim.y) * rows_side) {
    int rem = static_cast<int>(at);
    int64_t in = shard.in_off[last] + c, o = c;
    bool ok = true;
    for (int k = last - 1; k >= 0; --k) {
      const int x = rem % d.shard[k];
      rem /= d.shard[k];
      in += (x + shard.in_off[k]) * d.in_stride[k];
      o += x * d.out_stride[k];
      ok = ok && x < shard.valid[k];
    }
    float v[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = 0.f;
    if (ok && c < shard.valid[last]) {
      auto part = [&](int p) { return __builtin_nontemporal_load((GSPMD_GLOBAL const vec_t*)((GSPMD_GLOBAL const float*)args->ptrs.p[p] + in)); };
      vec_t sum;
      for (int p = 0; p < n_partials; p += 4) {            // fixed ascending order: deterministic
        vec_t g[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (p + q < n_partials) g[q] = part(p + q);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (p + q < n_partials) sum = p + q == 0 ? g[q] : sum + g[q];
      }
#pragma unroll
      for (int j = 0; j < VEC; ++j) v[j] = (c + j < shard.valid[last]) ? apply_epilogue(sum[j], epilogue) : 0.f;
    }
    if constexpr (VEC == 4) {
      f32x4 res;
      res.x = v[0]; res.y = v[1]; res.z = v[2]; res.w = v[3];
      store_stream4((TOut*)out + o, res);
    } else if constexpr (sizeof(TOut) == 2) {
      out[o] = float_to_bf16(v[0]);
    } else {
      out[o] = v[0];
    }
  }
}

// ---------------------------------------------------------------------------------------
// Shard <-> global copies (DynamicSlice / DynamicUpdateSlice of the appendix).
// ---------------------------------------------------------------------------------------
struct CopyDesc {
  int32_t rank;
  int64_t shard[kMaxRank];     // static shard shape
  int64_t valid[kMaxRank];
  int64_t sstride[kMaxRank];   // shard strides (elements)
  int64_t gstride[kMaxRank];   // global strides (elements), offset already folded into the base
};

// EXTRACT: shard[idx] = idx valid ? global[idx] : pad.   !EXTRACT: global[idx] = shard[idx] for valid idx.
// Element by element in 64-bit index arithmetic: for extents beyond the 31 bits of shard_move_kernel only.
template <typename T, bool EXTRACT>
__global__ __launch_bounds__(256) void shard_copy_kernel(CopyDesc d, const T* __restrict__ src,
                                                         T* __restrict__ dst, T pad, int64_t total) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    int64_t rem = i, so = 0, go = 0;
    bool ok = true;
    for (int k = d.rank - 1; k >= 0; --k) {
      const int64_t x = rem % d.shard[k];
      rem /= d.shard[k];
      so += x * d.sstride[k];
      go += x * d.gstride[k];
      ok = ok && (x < d.valid[k]);
    }
    if (EXTRACT) dst[so] = ok ? src[go] : pad;
    else if (ok) dst[go] = src[so];
  }
}

// ---------------------------------------------------------------------------------------
// Moves of boxes of a tensor: resharding (gather every dst shard from the src shards that own its elements), and the
// shard <-> global copies, which are the same with one src buffer.
// ---------------------------------------------------------------------------------------

// n / d for 0 <= n < 2^31 and 1 <= d < 2^31 without a division: q = (n * mul) >> 32 >> shift, mul = 2^(32 + shift) / d
// rounded up; exact because the rounding error n * (mul * d - 2^(32 + shift)) stays below 2^(32 + shift).
struct FastDiv {
  uint32_t mul, shift;           // d == 1: mul 0, shift 0 and the quotient is n itself
};
__host__ inline FastDiv fast_div(uint32_t d) {
  if (d <= 1) return FastDiv{0u, 0u};
  uint32_t s = 0;
  while ((uint64_t(2) << s) < d) ++s;                       // 2^s < d <= 2^(s+1)
  return FastDiv{static_cast<uint32_t>(((uint64_t(1) << (32 + s)) + d - 1) / d), s};
}
__host__ __device__ __forceinline__ uint32_t div_by(uint32_t n, FastDiv f) {
  return f.mul ? static_cast<uint32_t>((static_cast<uint64_t>(n) * f.mul) >> 32) >> f.shift : n;
}

// What all dst boxes of a move have in common.
struct MoveShape {
  int32_t rank;
  int32_t rows;                   // product of the dst box's extents except the last
  int32_t shard[kMaxRank];        // dst box, static extents (everything in it is written)
  int32_t src_per[kMaxRank];      // static shard size of src along each dimension
  int32_t pos_stride[kMaxRank];   // mesh-position stride of the mesh dimension src splits this dimension on (0 if none)
  FastDiv div_shard[kMaxRank], div_per[kMaxRank];   // by shard[k], by src_per[k]
  int64_t dst_stride[kMaxRank];
  int64_t src_stride[kMaxRank];
  uint32_t pad;                   // bits of the element written beyond the valid extents
  int32_t log_lanes;              // 2^log_lanes lanes walk along one row
  int32_t block_chunks;           // 16-byte chunks of a row that one workgroup takes
  int32_t unused;
};
struct MoveBox {                  // one per distinct dst buffer
  void* dst;
  int32_t valid[kMaxRank];        // valid extents: beyond them `pad` is written and nothing is read
  int32_t dst_off[kMaxRank];      // global index of the dst box's first element
  int32_t base_pos;               // mesh position contributed by the mesh dimensions src is not split on
  int32_t unused;
};
static_assert(sizeof(MoveBox) == 80, "device layout");

// 16 bytes of elements at an address that is only element-aligned: one 16-byte access (gfx950 takes any alignment
// for global loads and stores), where shards whose rows start anywhere used to go element by element.
template <typename T> struct ElementVec;
template <> struct ElementVec<bf16_bits> { typedef uint16_t type __attribute__((ext_vector_type(8), aligned(2))); };
template <> struct ElementVec<uint32_t> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };

// 2^log_lanes consecutive lanes walk along one dst row, 16 bytes at a time; grid.x covers the row in blocks of
// block_chunks chunks, grid.y strides over the rows, grid.z = dst buffer.  HBM bound: everything per row (where its
// elements are in src and dst) is worked out once per row and lane, everything per 16-byte chunk is one multiplication
// (which src shard owns its first element), and kMoveUnroll chunks' loads are issued before the first store.  Chunks
// are whole 16-byte blocks of dst; the loads take whatever alignment that leaves them, so any extent, offset and stride
// takes this path.  A chunk that crosses into another src shard or out of the row or its valid extent goes element by
// element.  Stores carry the non-temporal hint; loads do not (a misaligned load's line is wanted by the next lane's load
// too: with the hint 3.8 instead of 5.9 TB/s on the reshard below).
// Measured on one card against kernels that moved such rows element by element with divisions: 6000 x 10000 bf16 between
// two shardings on a 2 x 4 mesh (240 MB, rows of 2500 and 5000) 1.7 -> 6.8 TB/s; 1000000 x 24 0.2 -> 2.3; aligned AllGather of 537 MB
// 5.8 -> 8.2 (repeated calls, partly from the memory-side cache); cutting a 16384 x 8192 shard 1.6 -> 8.2; cutting
// 3000 x 2500 of 6000 x 10000 (30 MB) 20.3 -> 7.7 us.
constexpr int kMoveUnroll = 4;       // (8: 231 us, 2: 209, 1: 212 for the 17 moves that take 196 with 4)
template <typename T, typename ShapePtr, typename BoxPtr, typename SrcOf>
__device__ __forceinline__ void move_body(ShapePtr sp, BoxPtr bp, SrcOf src_of) {
  constexpr int V = 16 / static_cast<int>(sizeof(T));
  typedef typename ElementVec<T>::type Vec;
  typedef T AlignedVec __attribute__((ext_vector_type(16 / sizeof(T))));
  const auto& d = *sp;
  const auto& box = *bp;
  const int last = d.rank - 1;
  const int lanes = 1 << d.log_lanes, lane = threadIdx.x & (lanes - 1);
  const int per_group = blockDim.x >> d.log_lanes;                 // rows a workgroup walks side by side
  const int width = d.shard[last];
  const int valid_last = box.valid[last], off_last = box.dst_off[last], per_last = d.src_per[last], pos_last = d.pos_stride[last];
  const FastDiv div_last{d.div_per[last].mul, d.div_per[last].shift};
  GSPMD_GLOBAL T* const dst = (GSPMD_GLOBAL T*)box.dst;      // global (not flat) accesses
  const T pad = static_cast<T>(d.pad);
  for (uint32_t row = blockIdx.y * per_group + (threadIdx.x >> d.log_lanes); row < static_cast<uint32_t>(d.rows); row += gridDim.y * per_group) {
    uint32_t rem = row;
    int pos = box.base_pos;
    int64_t so = 0, o = 0;
    bool ok = true;
    for (int k = last - 1; k >= 0; --k) {
      const uint32_t q = div_by(rem, FastDiv{d.div_shard[k].mul, d.div_shard[k].shift});
      const uint32_t x = rem - q * static_cast<uint32_t>(d.shard[k]);
      rem = q;
      const uint32_t gk = static_cast<uint32_t>(box.dst_off[k]) + x;
      const uint32_t chunk = div_by(gk, FastDiv{d.div_per[k].mul, d.div_per[k].shift});
      pos += static_cast<int>(chunk) * d.pos_stride[k];
      so += static_cast<int64_t>(gk - chunk * static_cast<uint32_t>(d.src_per[k])) * d.src_stride[k];
      o += static_cast<int64_t>(x) * d.dst_stride[k];
      ok = ok && static_cast<int>(x) < box.valid[k];
    }
    const int row_valid = ok ? valid_last : 0;                     // columns of this row that come from src
    auto from = [&](int c) -> GSPMD_GLOBAL const T* {                           // src address of column c of the row, c < row_valid
      const uint32_t gl = static_cast<uint32_t>(off_last) + static_cast<uint32_t>(c);
      const uint32_t chunk = div_by(gl, div_last);
      return src_of(pos + static_cast<int>(chunk) * pos_last) + so + (gl - chunk * static_cast<uint32_t>(per_last));
    };
    // chunk i of the row holds columns [i V - mis, (i + 1) V - mis): whole chunks are aligned in dst, so every line of dst
    // is written by one wave-instruction or two consecutive ones; loads take whatever alignment is left
    const int mis = static_cast<int>((reinterpret_cast<uintptr_t>(dst + o) / sizeof(T)) & (V - 1));
    const int chunks = (width + mis + V - 1) / V, stop = min(chunks, static_cast<int>(blockIdx.x + 1) * d.block_chunks);
    for (int i0 = blockIdx.x * d.block_chunks + lane; i0 < stop; i0 += lanes * kMoveUnroll) {
      Vec v[kMoveUnroll];
      bool whole[kMoveUnroll];
#pragma unroll
      for (int u = 0; u < kMoveUnroll; ++u) {
        const int i = i0 + u * lanes, c = i * V - mis;
        whole[u] = false;
        if (i >= stop || c < 0 || c + V > width) continue;
        if (c >= row_valid) {
          v[u] = Vec(pad);
          whole[u] = true;
        } else if (c + V <= row_valid) {
          const uint32_t gl = static_cast<uint32_t>(off_last) + static_cast<uint32_t>(c);
          const uint32_t chunk = div_by(gl, div_last);
          const uint32_t local = gl - chunk * static_cast<uint32_t>(per_last);
          if (local + V <= static_cast<uint32_t>(per_last)) {
            GSPMD_GLOBAL const T* s = src_of(pos + static_cast<int>(chunk) * pos_last) + so + local;
            v[u] = *(GSPMD_GLOBAL const Vec*)s;
            whole[u] = true;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kMoveUnroll; ++u) {
        const int i = i0 + u * lanes, c = i * V - mis;
        if (whole[u]) {
          __builtin_nontemporal_store(v[u], (GSPMD_GLOBAL AlignedVec*)(dst + o + c));
        } else if (i < stop) {             // cut by an end of the row, the valid extent or a src shard: element by element
          T e[V];
#pragma unroll
          for (int j = 0; j < V; ++j) e[j] = (c + j >= 0 && c + j < row_valid) ? *from(c + j) : pad;
#pragma unroll
          for (int j = 0; j < V; ++j) if (c + j >= 0 && c + j < width) dst[o + c + j] = e[j];
        }
      }
    }
  }
}

// Tables small enough to travel as kernel arguments (no upload): up to kInlineReshardSrc partitions and
// kInlineReshardDescs distinct dst buffers; larger ones are read from device memory (`boxes` non-null).
constexpr int kInlineReshardSrc = 64, kInlineReshardDescs = 32;
struct InlineReshard {
  MoveShape shape;
  const void* src[kInlineReshardSrc];
  MoveBox d[kInlineReshardDescs];
};
static_assert(sizeof(InlineReshard) + 2 * sizeof(void*) <= 4096, "kernel arguments");

template <typename T>
__global__ __launch_bounds__(256) void reshard_kernel(const InlineReshard inl, const MoveBox* __restrict__ boxes,
                                                      const void* const* __restrict__ src_by_pos) {
  const GSPMD_KERNARG InlineReshard* in_args = first_kernel_argument<InlineReshard>();
  if (boxes) {
    move_body<T>(&in_args->shape, boxes + blockIdx.z, [=](int pos) { return (GSPMD_GLOBAL const T*)src_by_pos[pos]; });
  } else {
    // the table through LDS: a lane's own entry comes back in a tenth of a memory access's time
    __shared__ const void* table[kInlineReshardSrc];
    if (threadIdx.x < kInlineReshardSrc) table[threadIdx.x] = in_args->src[threadIdx.x];
    __syncthreads();
    const void* const* lds = table;
    move_body<T>(&in_args->shape, &in_args->d[blockIdx.z], [=](int pos) { return (GSPMD_GLOBAL const T*)lds[pos]; });
  }
}

// One box, one src buffer: a shard cut from a tensor, or put back into one.
struct ShardCopy {
  MoveShape shape;
  const void* src;
  MoveBox box;
};
template <typename T>
__global__ __launch_bounds__(256) void shard_move_kernel(const ShardCopy copy) {
  const GSPMD_KERNARG ShardCopy* in_args = first_kernel_argument<ShardCopy>();
  GSPMD_GLOBAL const T* const src = (GSPMD_GLOBAL const T*)in_args->src;
  move_body<T>(&in_args->shape, &in_args->box, [=](int) { return src; });
}

}  // namespace gspmd
