// Scheme U's compressors that keep the tensor on the chip, float32 input.
#include "uniform_chip_kernels.hpp"

namespace accept {

template hipError_t launch_held<float>(const accept_desc&, const UPlan&, const float*, float*, uint32_t*, ChipMail*, int, hipStream_t);
template hipError_t launch_channels<float>(const accept_desc&, const UPlan&, const float*, float*, uint32_t*, ChipMail*, int, hipStream_t);
template hipError_t launch_whole<float>(const accept_desc&, const UPlan&, const float*, float*, uint32_t*, ChipMail*, int, hipStream_t);

}  // namespace accept
