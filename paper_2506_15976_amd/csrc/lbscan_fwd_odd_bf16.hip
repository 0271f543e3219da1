// Forward kernels (wave tiles) for rows that start at odd elements, bf16 storage.
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_fwd_wave.inc"

namespace lbscan {
hipError_t launch_fwd_odd_bf16(const FwdParams& p, hipStream_t stream)
{
    return launch_fwd_t<bf16_t, Rows::odd>(p, stream);
}
}  // namespace lbscan
