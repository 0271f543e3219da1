// Forward kernels (wave tiles), bf16 storage.
#include "lbscan_device.h"
#include "lbscan_internal.h"
#include "lbscan_fwd_wave.inc"

namespace lbscan {
hipError_t launch_fwd_wave_bf16(const FwdParams& p, hipStream_t stream)
{
    return launch_fwd_t<bf16_t, Rows::aligned>(p, stream);
}
}  // namespace lbscan
