// Host-side launchers of the contraction kernels.  The kernels are compiled in sources of their own (one per operand
// layout), so that a build compiles them side by side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_basic.h"
#include "plan.h"

namespace gspmd {

constexpr int kMaxDevices = 64;

// One launch of a bf16 contraction kernel over `tiles` workgroups.
struct MfmaLaunch {
  const InlineProblems* inl;             // table that travels in the kernel arguments (tab null), or
  const Problem* tab;                    // table in device memory
  int n_prob, tiles, epilogue;
  float* join_partials;                  // joined problems: slots and arrival counters
  uint32_t* join_counters;
  unsigned long long* timeline;
  int timeline_records;
  bool spread = false;                   // dot_split_kernel: tiles in spread_tile's order
  bool past = false;                     // dot_mid_kernel: bf16 outputs past all caches
};

// `staged`: an operand does not take direct loads, both are loaded at element alignment through registers
template <int LAYOUT>
bool launch_dot_mfma_layout(const MfmaLaunch& l, int32_t out_dtype, bool staged, hipStream_t stream);

#ifndef GSPMD_TU_LAYOUT     // not where one layout is compiled
inline bool launch_dot_mfma(const MfmaLaunch& l, int32_t layout, int32_t out_dtype, bool staged, hipStream_t stream) {
  switch (layout & 3) {
    case 0: return launch_dot_mfma_layout<0>(l, out_dtype, staged, stream);
    case 1: return launch_dot_mfma_layout<1>(l, out_dtype, staged, stream);
    case 2: return launch_dot_mfma_layout<2>(l, out_dtype, staged, stream);
    default: return launch_dot_mfma_layout<3>(l, out_dtype, staged, stream);
  }
}
#endif

// One launch of dot_split_kernel in tiles of 16 * row_blocks rows (1, 2 or 4 blocks) x 16 * col_blocks columns (4; 2 with 1 or 2 row blocks; no joined
// problems).
constexpr int kSplitWaves = 8, kSplitThreads = 64 * kSplitWaves;
template <int LAYOUT>
bool launch_dot_split_layout(const MfmaLaunch& l, int32_t out_dtype, int row_blocks, int col_blocks, hipStream_t stream);

#ifndef GSPMD_TU_LAYOUT
inline bool launch_dot_split(const MfmaLaunch& l, int32_t layout, int32_t out_dtype, int row_blocks, int col_blocks, hipStream_t stream) {
  switch (layout & 3) {
    case 0: return launch_dot_split_layout<0>(l, out_dtype, row_blocks, col_blocks, stream);
    case 1: return launch_dot_split_layout<1>(l, out_dtype, row_blocks, col_blocks, stream);
    case 2: return launch_dot_split_layout<2>(l, out_dtype, row_blocks, col_blocks, stream);
    default: return launch_dot_split_layout<3>(l, out_dtype, row_blocks, col_blocks, stream);
  }
}
#endif

// One launch of dot_mid_kernel in 128 x 128 tiles.  `chain`: the launch has joined problems; the members of one output
// are consecutive in the table, in the order of summation, and only the first of them has tiles.  `staged`: operands through registers (no chain).
constexpr int kMidTile = 128, kMidThreads = 256;
constexpr int kMidAlone = 256;         // up to so many tiles a compute unit has one workgroup
template <int LAYOUT>
bool launch_dot_mid_layout(const MfmaLaunch& l, int32_t out_dtype, bool chain, bool staged, hipStream_t stream);

#ifndef GSPMD_TU_LAYOUT
inline bool launch_dot_mid(const MfmaLaunch& l, int32_t layout, int32_t out_dtype, bool chain, bool staged, hipStream_t stream) {
  switch (layout & 3) {
    case 0: return launch_dot_mid_layout<0>(l, out_dtype, chain, staged, stream);
    case 1: return launch_dot_mid_layout<1>(l, out_dtype, chain, staged, stream);
    case 2: return launch_dot_mid_layout<2>(l, out_dtype, chain, staged, stream);
    default: return launch_dot_mid_layout<3>(l, out_dtype, chain, staged, stream);
  }
}
#endif

// One launch of dot_pair_kernel in 256 x 128 tiles (no joined problems, direct loads, what is left of K in whole chunks).
constexpr int kPairRows = 256, kPairCols = 128;
template <int LAYOUT>
bool launch_dot_pair_layout(const MfmaLaunch& l, int32_t out_dtype, hipStream_t stream);

#ifndef GSPMD_TU_LAYOUT
inline bool launch_dot_pair(const MfmaLaunch& l, int32_t layout, int32_t out_dtype, hipStream_t stream) {
  switch (layout & 3) {
    case 0: return launch_dot_pair_layout<0>(l, out_dtype, stream);
    case 1: return launch_dot_pair_layout<1>(l, out_dtype, stream);
    case 2: return launch_dot_pair_layout<2>(l, out_dtype, stream);
    default: return launch_dot_pair_layout<3>(l, out_dtype, stream);
  }
}
#endif

}  // namespace gspmd
