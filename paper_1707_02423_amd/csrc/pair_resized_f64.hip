#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_resized_f64(int v) { return kernel_of<double, kModeResized>(v); }
}  // namespace cfsim
