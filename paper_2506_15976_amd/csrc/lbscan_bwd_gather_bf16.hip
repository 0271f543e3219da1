// Backward kernels, rows gathered in a scan order, bf16 storage (fp32 arithmetic).
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_bwd_wave.inc"

namespace lbscan {
hipError_t launch_bwd_gather_bf16(const BwdParams& p, hipStream_t stream)
{
    return launch_bwd_t<bf16_t, Rows::gathered>(p, stream);
}
}  // namespace lbscan
