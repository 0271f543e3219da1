// Forward kernels (wave tiles), fp32 storage.
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_fwd_wave.inc"

namespace lbscan {
hipError_t launch_fwd_wave_f32(const FwdParams& p, hipStream_t stream)
{
    return launch_fwd_t<float, Rows::aligned>(p, stream);
}
}  // namespace lbscan
