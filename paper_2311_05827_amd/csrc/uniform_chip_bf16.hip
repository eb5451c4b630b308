// Scheme U's compressors that keep the tensor on the chip, bfloat16 input.
#include "uniform_chip_kernels.hpp"

namespace accept {

template hipError_t launch_held<bf16_t>(const accept_desc&, const UPlan&, const bf16_t*, float*, uint32_t*, ChipMail*, int, hipStream_t);
template hipError_t launch_channels<bf16_t>(const accept_desc&, const UPlan&, const bf16_t*, float*, uint32_t*, ChipMail*, int, hipStream_t);
template hipError_t launch_whole<bf16_t>(const accept_desc&, const UPlan&, const bf16_t*, float*, uint32_t*, ChipMail*, int, hipStream_t);

}  // namespace accept
