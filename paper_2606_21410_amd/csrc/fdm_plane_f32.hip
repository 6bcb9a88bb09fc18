// Instantiations of the preconditioner's plane kernels, FP32.
#include "fdm_plane.h"

namespace cheb {
PLANE_INSTANCE(float, 1);
PLANE_INSTANCE(float, 2);
PLANE_INSTANCE(float, 3);
PLANE_INSTANCE(float, 4);
}  // namespace cheb
