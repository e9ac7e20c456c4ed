#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_damped_f64(int v) { return kernel_of<double, kModeDamped>(v); }
}  // namespace cfsim
