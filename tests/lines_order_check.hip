// store_lines (csrc/kernels_lines.h) as its kernels use it, without the Relu branch, whose blocks alone would keep the order: compiled, never run, by
// tests/test_lines_order.py.
#include "../paper_2105_04663_amd/csrc/kernels_lines.h"

namespace gspmd {

template <typename TOut, int BLOCKS, int AT_ONCE, LineStores STORES>
__global__ void check_kernel(Problem P, const float4_t* in) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  store_lines<TOut, BLOCKS, AT_ONCE, STORES>(smem, (GSPMD_GLOBAL TOut*)P.C, P, 0, 0, true, GSPMD_EPILOGUE_NONE, lane,
                                               [&](int i, int j) { return in[(i * 4 + j) * 64 + lane]; });
}
template __global__ void check_kernel<float, 4, 2, kLinesPlain>(Problem, const float4_t*);          // dot_mid_kernel
template __global__ void check_kernel<bf16_bits, 4, 4, kLinesPlain>(Problem, const float4_t*);
template __global__ void check_kernel<bf16_bits, 4, 4, kLinesThrough>(Problem, const float4_t*);
template __global__ void check_kernel<float, 8, 4, kLinesPlain>(Problem, const float4_t*);          // dot_pair_kernel
template __global__ void check_kernel<bf16_bits, 8, 8, kLinesPast>(Problem, const float4_t*);

}  // namespace gspmd
