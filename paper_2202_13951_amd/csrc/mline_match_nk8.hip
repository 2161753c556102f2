// m-line match-search kernel with 8 keys per lane (codes with n <= 512).
#include "mline_match_impl.h"

namespace orbg {
template hipError_t launch_mline_match_nk<8>(const MlineArgs& a, int grid, hipStream_t stream);
}  // namespace orbg
