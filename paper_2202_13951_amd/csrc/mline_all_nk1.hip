// Full (m-line) ORBGRAND decode of small batches with 1 key per lane (codes with n <= 64).
#include "mline_impl.h"

namespace orbg {
template hipError_t launch_mline_all_nk<1>(const MlineArgs& a, int grid, hipStream_t stream);
}  // namespace orbg
