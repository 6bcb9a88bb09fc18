// Matrix-core axis pass, FP64, row-block counts of 1, 2, 3 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(double, 1);
LINE_INSTANCE(double, 2);
LINE_INSTANCE(double, 3);
}  // namespace cheb
