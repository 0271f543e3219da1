// Backward kernels, rows gathered in a scan order, fp32 storage.
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_bwd_wave.inc"

namespace lbscan {
hipError_t launch_bwd_gather_f32(const BwdParams& p, hipStream_t stream)
{
    return launch_bwd_t<float, Rows::gathered>(p, stream);
}
}  // namespace lbscan
