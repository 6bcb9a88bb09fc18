// Instantiations of the preconditioner's plane kernels, FP64.
#include "fdm_plane.h"

namespace cheb {
PLANE_INSTANCE(double, 1);
PLANE_INSTANCE(double, 2);
PLANE_INSTANCE(double, 3);
PLANE_INSTANCE(double, 4);
}  // namespace cheb
