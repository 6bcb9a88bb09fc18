// Matrix-core axis pass, FP64, row-block counts of 4, 5 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(double, 4);
LINE_INSTANCE(double, 5);
}  // namespace cheb
