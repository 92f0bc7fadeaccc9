// Spot kernels of the forward model (wfs_forward_kernels.h) and of the sparse calibration
// (wfs_calib_kernels.h), subaperture sizes 2 to 6.
#include "wfs_calib_kernels.h"
#include "wfs_forward_kernels.h"

namespace wfs {
template hipError_t launch_fwd_ns<2>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<2>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<3>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<3>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<4>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<4>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<5>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<5>(const FwdParams&, const CalibParams&, hipStream_t);
template hipError_t launch_fwd_ns<6>(const FwdParams&, hipStream_t);
template hipError_t launch_calib_ns<6>(const FwdParams&, const CalibParams&, hipStream_t);
}  // namespace wfs
