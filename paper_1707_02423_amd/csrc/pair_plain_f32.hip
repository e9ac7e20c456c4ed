#include "pair_kernels.h"

namespace cfsim {
const void* pair_kernel_plain_f32(int v) { return kernel_of<float, kModePlain>(v); }
const void* strip_finish_f32() { return reinterpret_cast<const void*>(&strip_finish_kernel<float>); }
}  // namespace cfsim
