#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_plain_f64(int v) { return kernel_of<double, kModePlain>(v); }
}  // namespace cfsim
