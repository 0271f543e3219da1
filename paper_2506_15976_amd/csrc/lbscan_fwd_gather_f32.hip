// Forward kernels (wave tiles) that gather the tokens of a scan order, fp32 storage.
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_fwd_wave.inc"

namespace lbscan {
hipError_t launch_fwd_gather_f32(const FwdParams& p, hipStream_t stream)
{
    return launch_fwd_t<float, Rows::gathered>(p, stream);
}
}  // namespace lbscan
