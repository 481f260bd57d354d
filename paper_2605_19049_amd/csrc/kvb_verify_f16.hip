// kvb_verify_mfma_kernel for f16 inputs (fp32 and 16-bit records).
#include "kvb_verify_kernel.h"

namespace kvb_impl {

template void launch_verify_typed<f16_t, float>(int dk, const StepArgs &a, int blocks, hipStream_t stream);
template void launch_verify_typed<f16_t, f16_t>(int dk, const StepArgs &a, int blocks, hipStream_t stream);

}  // namespace kvb_impl
