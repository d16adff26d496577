// dot_pair_kernel for one operand layout (GSPMD_TU_LAYOUT, GSPMD_LAYOUT_* bits): compiled once per layout.
#include "kernels_pair.h"

namespace gspmd {

template bool launch_dot_pair_layout<GSPMD_TU_LAYOUT>(const MfmaLaunch& l, int32_t out_dtype, hipStream_t stream);

}  // namespace gspmd
