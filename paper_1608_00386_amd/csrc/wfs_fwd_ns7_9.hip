// Spot kernels of the forward model (wfs_forward_kernels.h) and of the sparse calibration
// (wfs_calib_kernels.h), subaperture sizes 7 to 9.
#include "wfs_calib_kernels.h"
#include "wfs_forward_kernels.h"

namespace wfs {
template hipError_t launch_fwd_ns<7>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<7>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<8>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<8>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<9>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<9>(const FwdParams&, const CalibParams&, hipStream_t);
}  // namespace wfs
