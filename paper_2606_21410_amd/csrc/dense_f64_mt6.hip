// Matrix-core axis pass, FP64, row-block counts of 6 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(double, 6);
}  // namespace cheb
