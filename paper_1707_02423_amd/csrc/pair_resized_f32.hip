#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_resized_f32(int v) { return kernel_of<float, kModeResized>(v); }
}  // namespace cfsim
