// The coarse tail and its reverse sweep, double cycles.
#include <hip/hip_runtime.h>

#include "tail.hpp"

namespace mgl {
MGL_TAIL_KERNELS(, double)
}  // namespace mgl
