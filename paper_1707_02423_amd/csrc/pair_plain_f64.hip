#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_plain_f64(int v) { return kernel_of<double, kModePlain>(v); }
const void* strip_finish_f64() { return reinterpret_cast<const void*>(&strip_finish_kernel<double>); }
}  // namespace cfsim
