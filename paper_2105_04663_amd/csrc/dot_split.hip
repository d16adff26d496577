// dot_split_kernel for one operand layout (GSPMD_TU_LAYOUT, GSPMD_LAYOUT_* bits): compiled once per layout.
#include "kernels_split.h"

namespace gspmd {

template bool launch_dot_split_layout<GSPMD_TU_LAYOUT>(const MfmaLaunch& l, int32_t out_dtype, int row_blocks, int col_blocks, hipStream_t stream);

}  // namespace gspmd
