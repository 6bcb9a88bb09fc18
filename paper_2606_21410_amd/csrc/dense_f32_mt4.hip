// Matrix-core axis pass, FP32, row-block counts of 4, 5 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(float, 4);
LINE_INSTANCE(float, 5);
}  // namespace cheb
