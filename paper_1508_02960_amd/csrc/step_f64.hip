// Step kernels for FP64 storage,
// instantiated here for the entry points of step_table.hpp.
#include <hip/hip_runtime.h>

#include "step_impl.hpp"

namespace lbm {
template const void* step_kernel_entry<double>(bool, int, bool, int, int);
template const void* batch_kernel_entry<double>(bool, int, int, int);
}  // namespace lbm
