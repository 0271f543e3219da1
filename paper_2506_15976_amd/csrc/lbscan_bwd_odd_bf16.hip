// Backward kernels, rows that start at odd elements, bf16 storage (fp32 arithmetic).
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_bwd_wave.inc"

namespace lbscan {
hipError_t launch_bwd_odd_bf16(const BwdParams& p, hipStream_t stream)
{
    return launch_bwd_t<bf16_t, Rows::odd>(p, stream);
}
}  // namespace lbscan
