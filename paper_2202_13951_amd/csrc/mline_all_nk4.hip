// Full (m-line) ORBGRAND decode of small batches with 4 keys per lane (codes with n <= 256).
#include "mline_impl.h"

namespace orbg {
template hipError_t launch_mline_all_nk<4>(const MlineArgs& a, int grid, hipStream_t stream);
}  // namespace orbg
