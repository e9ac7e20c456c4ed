#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_damped_f32(int v) { return kernel_of<float, kModeDamped>(v); }
}  // namespace cfsim
