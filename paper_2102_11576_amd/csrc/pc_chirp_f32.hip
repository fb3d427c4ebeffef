// Chirp-form sine-transform preconditioner with float internal arithmetic
// (explicit instantiations).
#include "pc_chirp.hpp"

namespace rsfde {
template hipError_t launch_cd_rows_fwd<float>(const CdDir&, const double*, const double*, float*, int, int,
                                           bool, hipStream_t);
template hipError_t launch_cd_cols<float>(const CdDir&, const float*, float*, float*, const double*,
                                       const double*, int, int, double, double, double, bool,
                                       hipStream_t);
template hipError_t launch_cd_rows_inv<float>(const CdDir&, const float*, const float*, const uint8_t*,
                                           double*, int, int, bool, hipStream_t);
template hipError_t launch_cd_dst_cols<float>(int, const float*, float*, const float*, float*, const void*,
                                           const void*, const void*, int, int, int, size_t,
                                           hipStream_t);
}  // namespace rsfde
