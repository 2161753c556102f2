// First-pass and match-search kernels with 4 keys per lane (codes with n <= 256).
#include "first_impl.h"

namespace orbg {
template hipError_t launch_match_nk<4>(const DecodeArgs& a, bool s32, bool listed, hipStream_t stream);
template hipError_t launch_first_nk<4>(const DecodeArgs& a, bool s32, hipStream_t stream);
}  // namespace orbg
