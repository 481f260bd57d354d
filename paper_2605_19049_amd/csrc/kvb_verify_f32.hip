// kvb_verify_mfma_kernel for fp32 inputs.
#include "kvb_verify_kernel.h"

namespace kvb_impl {

template void launch_verify_typed<float, float>(int dk, const StepArgs &a, int blocks, hipStream_t stream);

}  // namespace kvb_impl
