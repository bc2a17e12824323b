// The coarse tail and its reverse sweep, float cycles.
#include <hip/hip_runtime.h>

#include "tail.hpp"

namespace mgl {
MGL_TAIL_KERNELS(, float)
}  // namespace mgl
