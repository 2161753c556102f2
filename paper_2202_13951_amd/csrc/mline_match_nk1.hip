// m-line match-search kernel with 1 key per lane (codes with n <= 64).
#include "mline_match_impl.h"

namespace orbg {
template hipError_t launch_mline_match_nk<1>(const MlineArgs& a, int grid, hipStream_t stream);
}  // namespace orbg
