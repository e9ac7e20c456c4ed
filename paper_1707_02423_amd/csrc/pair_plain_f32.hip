#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_plain_f32(int v) { return kernel_of<float, kModePlain>(v); }
}  // namespace cfsim
