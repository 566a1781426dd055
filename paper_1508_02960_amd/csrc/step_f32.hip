// Step kernels for FP32 storage,
// instantiated here for the entry points of step_table.hpp.
#include <hip/hip_runtime.h>

#include "step_impl.hpp"

namespace lbm {
template const void* step_kernel_entry<float>(bool, int, bool, int, int);
template const void* batch_kernel_entry<float>(bool, int, int, int);
}  // namespace lbm
