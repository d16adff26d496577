// dot_mid_kernel for one operand layout (GSPMD_TU_LAYOUT, GSPMD_LAYOUT_* bits): compiled once per layout.
#include "kernels_mid.h"

namespace gspmd {

template bool launch_dot_mid_layout<GSPMD_TU_LAYOUT>(const MfmaLaunch& l, int32_t out_dtype, bool chain, bool staged, hipStream_t stream);

}  // namespace gspmd
