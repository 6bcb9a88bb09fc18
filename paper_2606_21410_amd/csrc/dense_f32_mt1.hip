// Matrix-core axis pass, FP32, row-block counts of 1, 2, 3 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(float, 1);
LINE_INSTANCE(float, 2);
LINE_INSTANCE(float, 3);
}  // namespace cheb
