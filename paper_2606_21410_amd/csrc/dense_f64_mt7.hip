// Matrix-core axis pass, FP64, row-block counts of 7 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(double, 7);
}  // namespace cheb
