// Single-axis slice kernels for detector sizes 75, 80, 81, 90, 96.
#include "axis_kernels.hpp"

namespace tomo {
const AxisSize kAxisSizesC[] = {axis_size<75>(), axis_size<80>(), axis_size<81>(), axis_size<90>(), axis_size<96>()};
const int kAxisSizesCCount = int(sizeof(kAxisSizesC) / sizeof(kAxisSizesC[0]));
}  // namespace tomo
