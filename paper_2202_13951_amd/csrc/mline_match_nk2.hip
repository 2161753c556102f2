// m-line match-search kernel with 2 keys per lane (codes with n <= 128).
#include "mline_match_impl.h"

namespace orbg {
template hipError_t launch_mline_match_nk<2>(const MlineArgs& a, int grid, hipStream_t stream);
}  // namespace orbg
