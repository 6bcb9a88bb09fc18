// Matrix-core axis pass, FP32, row-block counts of 6 (16 row pairs each).
#include "dense_launch.h"

namespace cheb {
LINE_INSTANCE(float, 6);
}  // namespace cheb
